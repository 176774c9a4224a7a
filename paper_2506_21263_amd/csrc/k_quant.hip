// QUANTIZE of Alg. 1 (symmetric per-group absmax quantiser, round-half-even) and the
// dequantise-and-average that stands in for the AllReduce of Alg. 2.
//
// One thread owns 4 consecutive elements, so a group of G elements is G/4 adjacent lanes of one
// wavefront and its absmax is a butterfly reduction over those lanes.  Integer decisions are
// taken in fp32 with an IEEE divide, one multiply and v_rndne, exactly as the payload is defined.
#include <type_traits>

#include "common.h"

namespace dlcx {

constexpr int kQThreads = 256;

template <int kLanes>  // lanes per group = group / 4
__device__ __forceinline__ float group_max(float a) {
#pragma unroll
    for (int off = kLanes >> 1; off >= 1; off >>= 1) a = fmaxf(a, __shfl_xor(a, off, 64));
    return a;
}

// Codes of four consecutive elements, packed as the payload holds them (16 bits of int4, 32 of int8), and the scale
// of their group.
template <int kQbits, int kLanes>
__device__ __forceinline__ uint32_t quantize4(const float4 &a, float &scale) {
    float amax = fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w)));
    amax = group_max<kLanes>(amax);
    constexpr float qmax = (float)((1 << (kQbits - 1)) - 1);
    float inv = 0.f;
    scale = 0.f;
    if (amax >= 0x1p-100f) {
        inv = qmax / amax;
        scale = amax / qmax;
    }
    const int c0 = (int)fminf(fmaxf(rintf(a.x * inv), -qmax), qmax);
    const int c1 = (int)fminf(fmaxf(rintf(a.y * inv), -qmax), qmax);
    const int c2 = (int)fminf(fmaxf(rintf(a.z * inv), -qmax), qmax);
    const int c3 = (int)fminf(fmaxf(rintf(a.w * inv), -qmax), qmax);
    constexpr uint32_t mask = kQbits == 4 ? 0xF : 0xFF;
    return (c0 & mask) | ((c1 & mask) << kQbits) | ((c2 & mask) << 2 * kQbits) | ((c3 & mask) << 3 * kQbits);
}
template <int kQbits>
__device__ __forceinline__ void store_codes(uint8_t *codes, int64_t v, uint32_t packed) {
    if (kQbits == 4) reinterpret_cast<uint16_t *>(codes)[v] = (uint16_t)packed;
    else reinterpret_cast<uint32_t *>(codes)[v] = packed;
}

// kSum: the input is S partial sums, added and written to sums[k] on the way (a pass of its own over
// them, 4 - 5 us behind every projection, cost as much as the quantiser itself).
template <int kQbits, int kLanes, bool kSum>
__global__ __launch_bounds__(kQThreads) void quantize_kernel(PtrPack<const float *> xs,
                                                             int64_t nvec,
                                                             PtrPack<uint8_t *> codes,
                                                             PtrPack<float *> scales, int64_t stride,
                                                             int S, int S_alt, const uint32_t *guard,
                                                             PtrPack<float *> sums) {
    const int k = blockIdx.y;
    const float *__restrict__ x = xs.p[k];
    const int64_t v = (int64_t)blockIdx.x * kQThreads + threadIdx.x;
    const bool live = v < nvec;  // whole groups are live or dead together
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (kSum) {
        if (live) {
            a = sum_partials(x, stride, split_count(S, S_alt, guard), v);
            reinterpret_cast<float4 *>(sums.p[k])[v] = a;
        }
    } else if (live) {
        a = reinterpret_cast<const float4 *>(x)[v];
    }
    float scale;
    const uint32_t packed = quantize4<kQbits, kLanes>(a, scale);
    if (!live) return;
    store_codes<kQbits>(codes.p[k], v, packed);
    if ((threadIdx.x & (kLanes - 1)) == 0) scales.p[k][v / kLanes] = scale;
}

// Mean of K decoded payloads of four elements: fp64 sum of the (exact) products code * scale in worker order, one
// rounding to fp32 at the end.
struct Mean4 {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    template <int kQbits>
    __device__ __forceinline__ void add(uint32_t w, float scale) {
        const double s = (double)scale;
        int c0, c1, c2, c3;
        if (kQbits == 4) {
            c0 = ((int)(w << 28)) >> 28;
            c1 = ((int)(w << 24)) >> 28;
            c2 = ((int)(w << 20)) >> 28;
            c3 = ((int)(w << 16)) >> 28;
        } else {
            c0 = ((int)(w << 24)) >> 24;
            c1 = ((int)(w << 16)) >> 24;
            c2 = ((int)(w << 8)) >> 24;
            c3 = ((int)w) >> 24;
        }
        a0 = fma((double)c0, s, a0);
        a1 = fma((double)c1, s, a1);
        a2 = fma((double)c2, s, a2);
        a3 = fma((double)c3, s, a3);
    }
    __device__ __forceinline__ float4 result(int K, double inv_k, int exact_inv) {
        if (exact_inv) {  // K a power of two: the reciprocal and the product are exact
            a0 *= inv_k; a1 *= inv_k; a2 *= inv_k; a3 *= inv_k;
        } else {
            const double kd = (double)K;
            a0 /= kd; a1 /= kd; a2 /= kd; a3 /= kd;
        }
        return make_float4((float)a0, (float)a1, (float)a2, (float)a3);
    }
};

// The quantiser and the mean of what it leaves, for callers that have all K workers' factors: a wavefront takes 256
// elements of one worker (of every kAvgWaves-th), the first one adds up what they decode to.  The same codes,
// scales and mean as the two kernels leave, without a launch and the payloads' way through memory between them: bound by
// latency at most sizes.  An outer step of one 512 x 512 matrix, which has two of them in its chain of launches, 74 - 79 us
// with a launch each, 61 in one; of an OPT-1.3B-like layer 1055 | 1015.  Above four workers a wavefront takes several of
// them one after the other, and one launch is still the shorter way for all of them.  P in bf16, us, two launches | one:
// 512 x 512 r = 8 K = 1 11.5 | 10.0, K = 8 15.1 | 12.2, K = 16 18.2 | 14.9; 8192 x 1024 r = 64 K = 4 40.4 | 37.1, K = 16
// 147 | 139; 8192 x 8192 r = 64 K = 8 416 | 392; 256 x 1280 r = 130 K = 16 37.5 | 34.4 (Q
// 35.8 | 29.7).
constexpr int kAvgWaves = 4;
template <int kQbits, int kLanes, bool kSum>
__global__ __launch_bounds__(64 * kAvgWaves) void quantize_average_kernel(
    int K, PtrPack<const float *> xs, int64_t nvec, PtrPack<uint8_t *> codes, PtrPack<float *> scales, int64_t stride,
    int S, int S_alt, const uint32_t *guard, PtrPack<float *> sums, double inv_k, int exact_inv,
    float *__restrict__ mean) {
    __shared__ uint32_t packed[DLCX_MAX_WORKERS][64];
    __shared__ float scale[DLCX_MAX_WORKERS][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t v = (int64_t)blockIdx.x * 64 + lane;
    const bool live = v < nvec;  // whole groups are live or dead together
    const int splits = kSum ? split_count(S, S_alt, guard) : 1;
    for (int k = wave; k < K; k += (int)(blockDim.x >> 6)) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live) {
            if constexpr (kSum) {
                a = sum_partials(xs.p[k], stride, splits, v);
                reinterpret_cast<float4 *>(sums.p[k])[v] = a;
            } else {
                a = reinterpret_cast<const float4 *>(xs.p[k])[v];
            }
        }
        float s;
        const uint32_t w = quantize4<kQbits, kLanes>(a, s);
        packed[k][lane] = w;
        scale[k][lane] = s;
        if (live) {
            store_codes<kQbits>(codes.p[k], v, w);
            if ((lane & (kLanes - 1)) == 0) scales.p[k][v / kLanes] = s;
        }
    }
    __syncthreads();
    if (wave != 0 || !live) return;
    Mean4 sum;
    for (int k = 0; k < K; ++k) sum.add<kQbits>(packed[k][lane], scale[k][lane]);  // workers in index order
    reinterpret_cast<float4 *>(mean)[v] = sum.result(K, inv_k, exact_inv);
}

template <int kQbits>
__global__ __launch_bounds__(kQThreads) void dequant_average_kernel(
    int K, PtrPack<const uint8_t *> codes, PtrPack<const float *> scales, int64_t nvec,
    int lanes_per_group, double inv_k, int exact_inv, float *__restrict__ out) {
    const int64_t v = (int64_t)blockIdx.x * kQThreads + threadIdx.x;
    if (v >= nvec) return;
    const int64_t g = v / lanes_per_group;
    Mean4 sum;
    for (int k = 0; k < K; ++k)  // workers in index order
        sum.add<kQbits>(kQbits == 4 ? reinterpret_cast<const uint16_t *>(codes.p[k])[v]
                                    : reinterpret_cast<const uint32_t *>(codes.p[k])[v],
                        scales.p[k][g]);
    reinterpret_cast<float4 *>(out)[v] = sum.result(K, inv_k, exact_inv);
}

template <int kQbits, bool kSum>
static int quantize_dispatch(int K, const PtrPack<const float *> &x, int64_t nvec, int group,
                             const PtrPack<uint8_t *> &codes, const PtrPack<float *> &scales,
                             const PartialSums &part, const PtrPack<float *> &sums, float *mean, hipStream_t st) {
    if (mean) {
        const dim3 grid((unsigned)ceil_div(nvec, 64)), block(64 * (K < kAvgWaves ? K : kAvgWaves));
        const double inv_k = 1.0 / (double)K;
        const int exact_inv = (K & (K - 1)) == 0;
        Timed timed(KID_QUANTIZE, st);
        auto launch = [&](auto lanes) {
            hipLaunchKernelGGL((quantize_average_kernel<kQbits, decltype(lanes)::value, kSum>), grid, block, 0, st, K, x,
                               nvec, codes, scales, part.stride, part.S, part.S_alt, part.guard, sums, inv_k, exact_inv,
                               mean);
            return check_launch("quantize_average");
        };
        switch (group) {
            case 16: return launch(std::integral_constant<int, 4>());
            case 32: return launch(std::integral_constant<int, 8>());
            case 64: return launch(std::integral_constant<int, 16>());
            case 128: return launch(std::integral_constant<int, 32>());
            case 256: return launch(std::integral_constant<int, 64>());
            default: return DLCX_EINVAL;
        }
    }
    const dim3 grid((unsigned)ceil_div(nvec, kQThreads), (unsigned)K);
    const dim3 block(kQThreads);
    Timed timed(KID_QUANTIZE, st);
    switch (group) {
        case 16: hipLaunchKernelGGL((quantize_kernel<kQbits, 4, kSum>), grid, block, 0, st, x, nvec, codes, scales, part.stride, part.S, part.S_alt, part.guard, sums); break;
        case 32: hipLaunchKernelGGL((quantize_kernel<kQbits, 8, kSum>), grid, block, 0, st, x, nvec, codes, scales, part.stride, part.S, part.S_alt, part.guard, sums); break;
        case 64: hipLaunchKernelGGL((quantize_kernel<kQbits, 16, kSum>), grid, block, 0, st, x, nvec, codes, scales, part.stride, part.S, part.S_alt, part.guard, sums); break;
        case 128: hipLaunchKernelGGL((quantize_kernel<kQbits, 32, kSum>), grid, block, 0, st, x, nvec, codes, scales, part.stride, part.S, part.S_alt, part.guard, sums); break;
        case 256: hipLaunchKernelGGL((quantize_kernel<kQbits, 64, kSum>), grid, block, 0, st, x, nvec, codes, scales, part.stride, part.S, part.S_alt, part.guard, sums); break;
        default: return DLCX_EINVAL;
    }
    return check_launch("quantize");
}

int launch_quantize(int K, const PtrPack<const float *> &x, int64_t count, int qbits, int group,
                    const PtrPack<uint8_t *> &codes, const PtrPack<float *> &scales,
                    hipStream_t st, float *mean) {
    if (count == 0 || K == 0) return DLCX_OK;
    const int64_t nvec = count >> 2;
    const PtrPack<float *> none = {};
    if (qbits == 4)
        return quantize_dispatch<4, false>(K, x, nvec, group, codes, scales, PartialSums(), none, mean, st);
    return quantize_dispatch<8, false>(K, x, nvec, group, codes, scales, PartialSums(), none, mean, st);
}

int launch_sum_quantize(int K, const PartialSums &part, const PtrPack<float *> &sums,
                        int64_t count, int qbits, int group, const PtrPack<uint8_t *> &codes,
                        const PtrPack<float *> &scales, float *mean, hipStream_t st) {
    if (count == 0 || K == 0) return DLCX_OK;
    if (mean && count > (int64_t)1 << 31) {  // a thread for every element: a launch has less than 2^32
        int rc = launch_sum_quantize(K, part, sums, count, qbits, group, codes, scales, nullptr, st);
        if (rc != DLCX_OK) return rc;
        PtrPack<const uint8_t *> cs;
        PtrPack<const float *> ss;
        for (int k = 0; k < K; ++k) {
            cs.p[k] = codes.p[k];
            ss.p[k] = scales.p[k];
        }
        return launch_dequant_average(K, cs, ss, count, qbits, group, mean, st);
    }
    const int64_t nvec = count >> 2;
    if (part.S == 1 && part.guard == nullptr) {
        PtrPack<const float *> x;
        for (int k = 0; k < K; ++k) x.p[k] = sums.p[k];
        return launch_quantize(K, x, count, qbits, group, codes, scales, st, mean);
    }
    if (qbits == 4)
        return quantize_dispatch<4, true>(K, part.slabs, nvec, group, codes, scales, part, sums, mean, st);
    return quantize_dispatch<8, true>(K, part.slabs, nvec, group, codes, scales, part, sums, mean, st);
}

int launch_dequant_average(int K, const PtrPack<const uint8_t *> &codes,
                           const PtrPack<const float *> &scales, int64_t count, int qbits,
                           int group, float *mean_out, hipStream_t st) {
    if (count == 0) return DLCX_OK;
    const int64_t nvec = count >> 2;
    const dim3 grid((unsigned)ceil_div(nvec, kQThreads));
    const double inv_k = 1.0 / (double)K;
    const int exact_inv = (K & (K - 1)) == 0;
    Timed timed(KID_DEQUANT_AVG, st);
    if (qbits == 4)
        hipLaunchKernelGGL(dequant_average_kernel<4>, grid, dim3(kQThreads), 0, st, K, codes,
                           scales, nvec, group / 4, inv_k, exact_inv, mean_out);
    else
        hipLaunchKernelGGL(dequant_average_kernel<8>, grid, dim3(kQThreads), 0, st, K, codes,
                           scales, nvec, group / 4, inv_k, exact_inv, mean_out);
    return check_launch("dequant_average");
}

}  // namespace dlcx
