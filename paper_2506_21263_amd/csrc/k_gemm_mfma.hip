// Rank-r products of the low-rank compressor on the bf16 matrix cores of gfx950
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation).
//
// Every fp32 operand is split into NS bf16 pieces, x = x0 + x1 (+ x2), each piece the bf16
// rounding of what the earlier pieces left over, and a product a*b is the sum of the piece
// products whose weight is not below the last piece:
//     NS = 2 (DLCX_MMA_BF16):  a0b0 + a0b1 + a1b0               error ~ 2^-17 per product
//     NS = 3 (DLCX_MMA_F32):   + a1b1 + a0b2 + a2b0             error ~ 2^-24 per product
// so the matrix cores run 3 or 6 bf16 instructions per 32x32x16 block.  At the ranks of interest
// the products are bound by the HBM stream of delta (4 bytes per element against 6r or 12r
// flops), not by the matrix cores, which is why the extra instructions are affordable; the native
// fp32 MFMA would cost 16 instruction issues of twice the latency for the same block.
//
// Operand layout of v_mfma_f32_32x32x16_bf16 (D = A B + C, A is 32 x 16, B is 16 x 32):
//   lane l holds A[l % 32][8 (l / 32) + e] and B[8 (l / 32) + e][l % 32], e = 0..7 (16 bytes);
//   D[i][j] is in lane j + 32 ((i / 4) % 2), register (i % 4) + 4 (i / 8).
// The small operand of every product (the basis, or both factors of the reconstruction) is first
// repacked ("fragments") so that a wavefront fetches one 32 x 16 operand block of one piece as
// 1 KB of consecutive memory; fragments are read straight from L2 into registers.  The big
// operand delta is staged through LDS (P phase, reduction along a row) or loaded straight into
// the operand layout with 128-byte row segments (Q phase, reduction down a column).
//
// Kernels in this file:
//   pack_kcontig_kernel, pack_f16_kernel, pack_sweep_kernel   fragments of a basis, of both forms
//                                                 of a basis, of all operands of a sweep
//   project_p_ws_kernel, project_q_ws_kernel      projections with producer and consumer
//                                                 wavefronts
//   project_p_one_kernel, project_q_one_kernel    projections at r <= 32 (P where it is the faster
//                                                 one, Q of three pieces), every wavefront does
//                                                 everything
//   reconstruct_mfma_kernel                       Delta_hat tile by tile with the elementwise
//                                                 steps of Alg. 2 fused in (any rank)
//   round_mfma_kernel                             the same plus the P phase of the next
//                                                 compression: the benchmark's hot kernel (r <= 64)
// Two things learnt on this hardware shape all of them.  A wavefront's loads return in order, so
// a wait for something needed soon (a fragment from L2) also waits for everything requested
// before it (delta from HBM, needed much later): requests are issued in the order of need, or
// the two kinds of load are given to different wavefronts.  And a load behind a per-lane
// condition cuts the loop into small blocks that the compiler schedules one by one: lanes
// outside the matrix read a valid address instead and the value is dropped.
#include <type_traits>

#include "common.h"

namespace dlcx {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kW = 256;  // threads per workgroup (4 wavefronts)

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {  // round-to-nearest-even
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ uint32_t pack_f16x2(float a, float b) {  // round-to-nearest-even
    typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, f16x2_t));
}

// pieces of the pair (a, b): out[h] holds piece h of a in its low half, of b in its high half.
// NS == 1 is the fp16 form of an operand: one piece, the fp16 rounding of the value (the caller
// has scaled it into fp16's range by a power of two).
template <int NS>
__device__ __forceinline__ void split2(float a, float b, uint32_t (&out)[NS]) {
    if constexpr (NS == 1) {
        out[0] = pack_f16x2(a, b);
        return;
    }
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        const uint32_t p = pack_bf16x2(a, b);
        out[h] = p;
        if (h + 1 < NS) {
            a -= __uint_as_float(p << 16);
            b -= __uint_as_float(p & 0xFFFF0000u);
        }
    }
}

// 8 consecutive-k values -> NS operand registers (uint4 = 8 bf16)
template <int NS>
__device__ __forceinline__ void split8(const float (&x)[8], uint4 (&out)[NS]) {
    uint32_t p[4][NS];
#pragma unroll
    for (int q = 0; q < 4; ++q) split2<NS>(x[2 * q], x[2 * q + 1], p[q]);
#pragma unroll
    for (int h = 0; h < NS; ++h) out[h] = make_uint4(p[0][h], p[1][h], p[2][h], p[3][h]);
}

__device__ __forceinline__ f32x16_t mfma(const uint4 &a, const uint4 &b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

template <int NS>
__device__ __forceinline__ void mfma_split(const uint4 (&a)[NS], const uint4 (&b)[NS],
                                           f32x16_t &c) {
    if constexpr (NS == 1) {  // one fp16 product
        typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a[0]),
                                                   __builtin_bit_cast(f16x8_t, b[0]), c, 0, 0, 0);
        return;
    }
    if (NS == 3) {  // smallest terms first
        c = mfma(a[2], b[0], c);
        c = mfma(a[0], b[2], c);
        c = mfma(a[1], b[1], c);
    }
    if (NS >= 2) {
        c = mfma(a[1], b[0], c);
        c = mfma(a[0], b[1], c);
    }
    c = mfma(a[0], b[0], c);
}

// The same with the products of the smaller pieces in an accumulator of their own (kApart), added to
// `c` at the end of the sum by the caller.  They are 2^-8 of the others or less: c is rounded once per
// 16 terms instead of NS (NS + 1) / 2 times, and in a long sum that rounding is the fp32 error.
template <int NS, bool kApart>
__device__ __forceinline__ void mfma_split_sum(const uint4 (&a)[NS], const uint4 (&b)[NS],
                                               f32x16_t &c, f32x16_t &small) {
    if constexpr (!kApart) {
        mfma_split<NS>(a, b, c);
    } else {
        if (NS == 3) {
            small = mfma(a[2], b[0], small);
            small = mfma(a[0], b[2], small);
            small = mfma(a[1], b[1], small);
        }
        small = mfma(a[1], b[0], small);
        small = mfma(a[0], b[1], small);
        c = mfma(a[0], b[0], c);
    }
}

// row of D held in register v of lane `lane`
__device__ __forceinline__ int d_row(int v, int lane) {
    return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
}

// Accesses to the big streams (delta, theta_l, theta, v), each touched once per sweep: marked
// non-temporal so that they do not displace the fragments and one another in the caches.
typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t nt_u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float4 stream_load4(const float *p) {
    const nt_f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f32x4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 stream_load2(const void *p) {
    const nt_u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x2 *>(p));
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ void stream_store4(float *p, const float4 &a) {
    const nt_f32x4 v = {a.x, a.y, a.z, a.w};
    __builtin_nontemporal_store(v, reinterpret_cast<nt_f32x4 *>(p));
}

// ---------------------------------------------------------------------------------------------
// Fragment packing.
// ---------------------------------------------------------------------------------------------
// src is nrows x L with the reduction index contiguous (a basis: Q_in is r x n, P_hat is r x m).
// Fragment (s, rb, h): rows rb*32 .. +32, reduction indices s*16 .. +16, piece h, at
// frags[((s * RB + rb) * NS + h) * 64 + lane].  Rows >= nrows and indices >= L are zero.
struct KContig {
    const float *src;
    int nrows;
    int64_t L;
    int RB;
    int64_t KS;
    uint4 *frags;
    __host__ __device__ int64_t count() const { return KS * RB; }
};
__device__ __forceinline__ bool load_kcontig(const KContig &p, int64_t f, int lane, float (&x)[8]) {
    const int row = (int)(f % p.RB) * 32 + (lane & 31);
    const int64_t k0 = f / p.RB * 16 + (lane >> 5) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = 0.f;
    if (row >= p.nrows || k0 >= p.L) return false;  // L is a multiple of 8
    const float4 a = *reinterpret_cast<const float4 *>(p.src + (int64_t)row * p.L + k0);
    const float4 b = *reinterpret_cast<const float4 *>(p.src + (int64_t)row * p.L + k0 + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    return true;
}
template <int NS>
__device__ __forceinline__ void store_frags(uint4 *frags, int64_t f, int lane, const float (&x)[8]) {
    uint4 out[NS];
    split8<NS>(x, out);
#pragma unroll
    for (int h = 0; h < NS; ++h) frags[(f * NS + h) * 64 + lane] = out[h];
}

template <int NS>
__global__ __launch_bounds__(kW) void pack_kcontig_kernel(KContig p) {
    const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (f >= p.count()) return;
    float x[8];
    load_kcontig(p, f, lane, x);
    store_frags<NS>(p.frags, f, lane, x);
}

// Both forms a DLCX_MMA_F16 projection keeps ready, from one read of the basis: two bf16 pieces for
// the stand-by and one fp16 piece of the rows scaled by row_scale (powers of two: exact).
__global__ __launch_bounds__(kW) void pack_f16_kernel(KContig p, uint4 *__restrict__ frags_f16,
                                                      const float *__restrict__ row_scale) {
    const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (f >= p.count()) return;
    float x[8];
    const bool in = load_kcontig(p, f, lane, x);
    store_frags<2>(p.frags, f, lane, x);
    const float sc = in ? row_scale[(int)(f % p.RB) * 32 + (lane & 31)] : 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] *= sc;
    store_frags<1>(frags_f16, f, lane, x);
}

// The fp16 form of a projection (NS == 1) needs its operands inside fp16's range.  delta is
// multiplied by 2^kF16DeltaShift, which is safe while the largest |delta| of the launch lies in
// [2^-14, 15.99) (the kernel records it; outside that window the bf16 kernel redoes the launch).
// Every row of the basis (one factor column) gets its own power of two that puts its largest
// entry into [2^7, 2^8): in_scale[c] for the fragments, out_scale[c] = 2^-kF16DeltaShift /
// in_scale[c] for the result, so that scaling is exact and invisible.  Workgroup c handles row c;
// workgroup 0 also clears the launch's record of the largest |delta|.
constexpr int kF16DeltaShift = 12;
__global__ __launch_bounds__(kW) void basis_scale_kernel(const float *__restrict__ src, int64_t L,
                                                         float *__restrict__ in_scale,
                                                         float *__restrict__ out_scale,
                                                         uint32_t *__restrict__ amax_record) {
    __shared__ float red[kW];
    const int c = blockIdx.x;
    float a = 0.f;
    for (int64_t i = threadIdx.x * 4; i < L; i += kW * 4) {  // L is a multiple of 8
        const float4 v = *reinterpret_cast<const float4 *>(src + (int64_t)c * L + i);
        a = fmaxf(fmaxf(a, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
    }
    red[threadIdx.x] = a;
    __syncthreads();
    for (int s = kW / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float amax = red[0];
        int e = 0;
        if (amax > 0.f && amax < 3.0e38f) e = 7 - ilogbf(amax);
        e = e < -100 ? -100 : (e > 100 ? 100 : e);
        in_scale[c] = ldexpf(1.f, e);
        out_scale[c] = ldexpf(1.f, -e - kF16DeltaShift);
        if (c == 0) *amax_record = 0u;
    }
}

// largest |x| over a wavefront, then one atomic per wavefront (bit patterns of non-negative
// floats order like the floats)
__device__ __forceinline__ void record_amax(float a, uint32_t *record) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a = fmaxf(a, __shfl_xor(a, off, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(record, __float_as_uint(a));
}

// src is r x L with the reduction index c strided (a factor used in the reconstruction).
// Fragment (xb, s, h): positions xb*32 .. +32 along L, reduction indices s*16 .. +16, at
// frags[((xb * KS + s) * NS + h) * 64 + lane].
struct KStrided {
    const float *src;
    int r;
    int64_t L;
    int KS;
    int64_t XB;
    uint4 *frags;
    __host__ __device__ int64_t count() const { return XB * KS; }
};
template <int NS>
__device__ __forceinline__ void pack_kstrided(const KStrided &p, int64_t f, int lane) {
    const int64_t x0 = f / p.KS * 32 + (lane & 31);
    const int c0 = (int)(f % p.KS) * 16 + (lane >> 5) * 8;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        x[e] = (x0 < p.L && c0 + e < p.r) ? p.src[(int64_t)(c0 + e) * p.L + x0] : 0.f;
    store_frags<NS>(p.frags, f, lane, x);
}

// Everything a sweep needs packed, in one launch (three of them in a row cost 4 - 5 us each, whatever
// the size): the fragments of the basis (if any), then those of both factors of the reconstruction.
template <int NS>
__global__ __launch_bounds__(kW) void pack_sweep_kernel(KContig basis, KStrided p_hat, KStrided q_bar) {
    int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (f < basis.count()) {
        float x[8];
        load_kcontig(basis, f, lane, x);
        store_frags<NS>(basis.frags, f, lane, x);
        return;
    }
    f -= basis.count();
    if (f < p_hat.count()) {
        pack_kstrided<NS>(p_hat, f, lane);
        return;
    }
    f -= p_hat.count();
    if (f < q_bar.count()) pack_kstrided<NS>(q_bar, f, lane);
}

// ---------------------------------------------------------------------------------------------
// P phase:  P_k[i][c] = sum_j delta_k[i][j] Q_in[c][j].
// Workgroup: RB row blocks (32 RB rows) of delta, swept along its range of columns j in stages of 64
// (4 k-steps); A = basis fragments (M = c), B = delta from LDS (N = i): D[c][i].  A basis fragment
// serves RB / WR row blocks once it is in registers, so the fragment traffic per byte of delta
// falls with RB: at r = 256 it is 4 : 1 with 64 rows and 2 : 1 with 128.  A stage of matrix-core work
// is about as long as a round trip to HBM and a single wavefront per SIMD cannot hide one behind the
// other, so the workgroup has 8 wavefronts with two roles.  Wavefronts 4..7 (producers) stream delta: stage s
// lives in register set s & 1, is split into bf16 pieces and laid down in LDS buffer s & 1 one
// stage before it is used, and its set is refilled at once with stage s + 2, so that every
// request has two stages of time to come back.  Wavefronts 0..3 (consumers) own WC x WR blocks of
// the output, fetch their basis fragments through L2 two or four k-steps ahead (their load
// counter never waits for HBM) and keep the matrix cores busy on the buffer the producers filled
// last.  One
// LDS-only barrier per stage for all eight.  Loads past the matrix or past the last stage are
// clamped to a valid address and zeroed / never read, which keeps both loops free of branches.
// ---------------------------------------------------------------------------------------------
constexpr int kPPitch = 64 * 2 + 16;  // bytes per LDS row of one piece: 64 bf16 + pad

// Workgroup barrier for data exchanged through LDS: every LDS access of this wavefront has
// completed before it arrives, and the compiler moves no memory access across.  Global loads
// that are still outstanding (the next stage, already requested) are NOT waited for, which
// __syncthreads() would do.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr int kWs = 512;  // threads of the two-role workgroup

// NS == 1 is the fp16 form (one product per block instead of three): the producers multiply
// delta by 2^kF16DeltaShift and record its largest magnitude in *amax_record, the consumers undo
// the scales through out_scale.  `guard` (NS >= 2) makes the launch a stand-by: it returns at
// once if the fp16 launch before it saw its operands in range.
// Accumulators of the small products (mfma_split_sum) at 1 and 2 basis blocks, where the registers are
// there for the asking.  Error against fp64 of three pieces, 6528 x 5136 at r = 4: 4.5e-7, in one
// accumulator 1.1e-6; 8192 x 8192 r = 20 193 us either way.
template <int NS, int BLOCKS>
constexpr bool kApartP = NS >= 2 && BLOCKS <= 2;
// Accumulators that take the k-steps in turn, where a wavefront has one block: half as many roundings in
// each.  Error against fp64, 8192 x 8192 r = 20 three pieces 2.4e-7 (in one accumulator 4.7e-7), 8192 x
// 2048 r = 32 two pieces 4.2e-7 (4.7e-7); no difference in time.
// LONE: as many where it has two, if there are no two workgroups to a compute unit (registers).
template <int NS, int BLOCKS, bool LONE>
constexpr int kChainsP = NS >= 2 && BLOCKS <= (LONE ? 2 : 1) ? 2 : 1;
// Wavefronts to a SIMD that the registers have to leave room for: two workgroups to a compute unit at up to 4
// basis blocks, that is 128 registers.  Left to itself the compiler takes 130 for three of these kernels, and a
// workgroup has its unit to itself.  Two pieces, us with one | two to a unit: 28672 x 8192 four workers r = 100
// 943 | 884, r = 24 656 | 632; 8192 x 8192 r = 100 five workers 410 | 386, eight 503 | 483.  At ranks 33 .. 64
// it goes either way: 8192 x 2048 six workers r = 64 102 | 95, 28672 x 2048 two workers r = 40 105 | 99, but
// where few units get a second workgroup 8192 x 8192 five workers 283 | 313, 40960 x 8192 one 284 | 313.
template <int NS, int BLOCKS, bool LONE>
constexpr int kWavesP = NS <= 2 && BLOCKS <= 4 && !LONE ? 4 : 1;
template <int NS, int CBW, int WC, int WR, int RB, bool LONE, int kSets = 2>
__global__ __launch_bounds__(kWs, (kWavesP<NS, CBW * WC, LONE>)) void project_p_ws_kernel(
    PtrPack<const float *> deltas, const uint4 *__restrict__ afrags, PtrPack<float *> outs, int64_t m, int64_t n,
    int r, int64_t stages_per_wg, int64_t slab_stride, uint32_t *__restrict__ amax_record,
    const float *__restrict__ out_scale, const uint32_t *__restrict__ guard) {
    constexpr int CB = CBW * WC;
    constexpr int RBW = RB / WR;
    constexpr int kRows = 32 * RB;
    constexpr int kVec = kRows * 16 / kW;  // float4 per producer thread and stage
    static_assert(WC * WR == 4, "four consumer wavefronts");
    constexpr int kBuf = NS * kRows * kPPitch;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    if (guard != nullptr && f16_range_ok(*guard)) return;  // uniform over the launch
    const float *__restrict__ delta = deltas.p[blockIdx.y];
    float *__restrict__ out = outs.p[blockIdx.y] + (int64_t)blockIdx.z * slab_stride;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * kRows;
    const int64_t sfirst = (int64_t)blockIdx.z * stages_per_wg;  // of the matrix's stages of 64 columns
    const int64_t sleft = (n + 63) / 64 - sfirst;
    const int64_t nstages = stages_per_wg < sleft ? stages_per_wg : sleft;

    if (wave >= 4) {  // ---------------------------------------------------------- producers
        const int tid = threadIdx.x - kW;
        float amax = 0.f;  // NS == 1: largest |delta| this thread has laid down
        auto load_stage = [&](float4 (&set)[kVec], int64_t t) {
            const int64_t tc = t < nstages ? t : nstages - 1;
#pragma unroll
            for (int u = 0; u < kVec; ++u) {
                const int idx = tid + kW * u;
                const int row = idx >> 4, c4 = idx & 15;
                const int64_t j = (sfirst + tc) * 64 + c4 * 4;
                const bool ok = i0 + row < m && j < n;
                // the value of a clamped load is discarded when the stage is laid down, not
                // here: touching it now would wait for the request just made
                set[u] = stream_load4(ok ? delta + (i0 + row) * n + j : delta);
            }
        };
        auto store_stage = [&](const float4 (&set)[kVec], unsigned char *buf, int64_t t) {
#pragma unroll
            for (int u = 0; u < kVec; ++u) {
                const int idx = tid + kW * u;
                const int row = idx >> 4, c4 = idx & 15;
                const bool ok = i0 + row < m && (sfirst + t) * 64 + c4 * 4 < n;
                float4 x = make_float4(ok ? set[u].x : 0.f, ok ? set[u].y : 0.f,
                                       ok ? set[u].z : 0.f, ok ? set[u].w : 0.f);
                if constexpr (NS == 1) {
                    amax = fmaxf(fmaxf(amax, fmaxf(fabsf(x.x), fabsf(x.y))),
                                 fmaxf(fabsf(x.z), fabsf(x.w)));
                    constexpr float kUp = (float)(1 << kF16DeltaShift);
                    x = make_float4(x.x * kUp, x.y * kUp, x.z * kUp, x.w * kUp);
                }
                uint32_t lo[NS], hi[NS];
                split2<NS>(x.x, x.y, lo);
                split2<NS>(x.z, x.w, hi);
#pragma unroll
                for (int h = 0; h < NS; ++h)
                    *reinterpret_cast<uint2 *>(buf + (h * kRows + row) * kPPitch + c4 * 8) =
                        make_uint2(lo[h], hi[h]);
            }
        };
        // one step: lay down stage `stage` (held in `set`) for the consumers' next iteration
        // while they work on the stage before it, then refill the set kSets stages further on
        // (four sets measured no faster than three at best)
        auto step = [&](float4 (&set)[kVec], int64_t stage, bool refill) {
            store_stage(set, lds + (stage & 1) * kBuf, stage);
            if (refill) load_stage(set, stage + kSets);
            lds_barrier();
            // nothing of the next step moves above the barrier: splitting its set earlier would
            // wait for requests that are younger than they should be
            __builtin_amdgcn_sched_barrier(0);
        };
        float4 set[kSets][kVec];
#pragma unroll
        for (int s = 0; s < kSets; ++s) load_stage(set[s], s);
        step(set[0], 0, true);
        // kSets stages per trip, no way round the later ones inside the loop: the compiler's wait
        // counts at the loop head then see one order of outstanding requests only.
        int64_t t = 0;
        for (; t + kSets - 1 < nstages; t += kSets)
#pragma unroll
            for (int s = 1; s <= kSets; ++s) step(set[s % kSets], t + s, true);
        // what is left: the consumers' last iteration needs its barrier
#pragma unroll
        for (int s = 1; s < kSets; ++s)
            if (t + s <= nstages) step(set[s], t + s, false);
        if constexpr (NS == 1) record_amax(amax, amax_record);
        return;
    }
    // -------------------------------------------------------------------------------- consumers
    const int wc = wave % WC, wr = wave / WC;
    constexpr bool kApart = kApartP<NS, CBW * RBW>;
    constexpr int kTurns = kChainsP<NS, CBW * RBW, LONE>;
    f32x16_t acc[kTurns][CBW][RBW], small[kApart ? CBW : 1][kApart ? RBW : 1];
#pragma unroll
    for (int a = 0; a < CBW; ++a)
#pragma unroll
        for (int b = 0; b < RBW; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
#pragma unroll
                for (int t = 0; t < kTurns; ++t) acc[t][a][b][v] = 0.f;
                if constexpr (kApart) small[a][b][v] = 0.f;
            }
    // fragments of global k-step g (4 per stage) in ring position g % AD: requested two k-steps
    // ahead, or a whole stage ahead where that is at most 8 registers per position (one fp16
    // piece, or one basis block per wavefront).  There the matrix-core work of two k-steps is
    // shorter than a trip to L2 and the consumers, hence the stage barrier, waited for fragments:
    // 4 - 10 % on the kernel at rank 64, 4 - 7 % in the fp16 form at ranks 192 and 256.  With two
    // blocks of two bf16 pieces the matrix cores set the pace and the deeper ring gains nothing.
    constexpr int AD = CBW * NS <= 2 ? 4 : 2;
    uint4 a[AD][CBW][NS];
    const int64_t gmax = nstages * 4 - 1;
    auto load_frags = [&](int64_t g, int pos) {
        const int64_t gc = sfirst * 4 + (g < gmax ? g : gmax);
#pragma unroll
        for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
            for (int h = 0; h < NS; ++h)
                a[pos][cb][h] = afrags[((gc * CB + wc * CBW + cb) * NS + h) * 64 + lane];
    };
#pragma unroll
    for (int g = 0; g < AD; ++g) load_frags(g, g);
    lds_barrier();
    for (int64_t t = 0; t < nstages; ++t) {
        const unsigned char *buf = lds + (t & 1) * kBuf;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            uint4 b[RBW][NS];
#pragma unroll
            for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
                for (int h = 0; h < NS; ++h) {
                    const int row = (wr * RBW + rb) * 32 + (lane & 31);
                    b[rb][h] = *reinterpret_cast<const uint4 *>(
                        buf + (h * kRows + row) * kPPitch + ks * 32 + (lane >> 5) * 16);
                }
#pragma unroll
            for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
                for (int rb = 0; rb < RBW; ++rb)
                    mfma_split_sum<NS, kApart>(a[ks % AD][cb], b[rb], acc[ks % kTurns][cb][rb],
                                               small[kApart ? cb : 0][kApart ? rb : 0]);
            // requested here and nowhere later: AD k-steps of matrix-core work to come back
            load_frags(t * 4 + ks + AD, ks % AD);
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier();
    }
#pragma unroll
    for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if constexpr (kApart) acc[0][cb][rb][v] += small[cb][rb][v];
                if constexpr (kTurns == 2) acc[0][cb][rb][v] += acc[1][cb][rb][v];
            }
#pragma unroll
    for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
        for (int rb = 0; rb < RBW; ++rb) {
            const int64_t i = i0 + (wr * RBW + rb) * 32 + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int c = (wc * CBW + cb) * 32 + d_row(v, lane);
                if (c < r && i < m)
                    out[(int64_t)c * m + i] = NS == 1 ? acc[0][cb][rb][v] * out_scale[c] : acc[0][cb][rb][v];
            }
        }
}

// The same product with every wavefront doing everything, 64 rows per workgroup: wavefront (wk, wr) takes
// 32 rows and the k-steps 2 wk, 2 wk + 1 of every stage, the two halves are added at the end; basis
// fragments are requested a stage ahead and before the next stage of delta.  For one basis block, where the
// matrix cores have little to do: four such workgroups share a compute unit (two with three pieces) and
// even out what 128 rows at a time leave over.  Where it is used: p_plan.
constexpr int kOneRows = 64;
template <int NS>
__global__ __launch_bounds__(kW) void project_p_one_kernel(PtrPack<const float *> deltas,
                                                           const uint4 *__restrict__ afrags,
                                                           PtrPack<float *> outs, int64_t m,
                                                           int64_t n, int r) {
    constexpr int kVec = kOneRows * 16 / kW;  // float4 per thread and stage
    constexpr int kBuf = NS * kOneRows * kPPitch;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * kBuf];
    const float *__restrict__ delta = deltas.p[blockIdx.y];
    float *__restrict__ out = outs.p[blockIdx.y];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wk = wave & 1, wr = wave >> 1;
    const int64_t i0 = (int64_t)blockIdx.x * kOneRows;
    const int64_t nstages = (n + 63) / 64;
    f32x16_t acc, small;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = small[v] = 0.f;

    float4 pre[kVec];  // this thread's share of a stage: (row, 4 columns)
    auto load_stage = [&](int64_t t) {
#pragma unroll
        for (int u = 0; u < kVec; ++u) {
            const int idx = tid + kW * u;
            const int row = idx >> 4;
            const int64_t j = t * 64 + (idx & 15) * 4;
            pre[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i0 + row < m && j < n) pre[u] = stream_load4(delta + (i0 + row) * n + j);
        }
    };
    uint4 a[2][NS];
    auto load_frags = [&](uint4 (&dst)[2][NS], int64_t t) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int h = 0; h < NS; ++h)
                dst[ks][h] = afrags[((t * 4 + wk * 2 + ks) * NS + h) * 64 + lane];
    };
    load_frags(a, 0);
    load_stage(0);
    for (int64_t t = 0; t < nstages; ++t) {
        unsigned char *buf = lds + (t & 1) * kBuf;
#pragma unroll
        for (int u = 0; u < kVec; ++u) {
            const int idx = tid + kW * u;
            uint32_t lo[NS], hi[NS];
            split2<NS>(pre[u].x, pre[u].y, lo);
            split2<NS>(pre[u].z, pre[u].w, hi);
#pragma unroll
            for (int h = 0; h < NS; ++h)
                *reinterpret_cast<uint2 *>(buf + (h * kOneRows + (idx >> 4)) * kPPitch + (idx & 15) * 8) =
                    make_uint2(lo[h], hi[h]);
        }
        // fragments before delta: waiting for them later does not wait for that stage as well
        uint4 an[2][NS];
        if (t + 1 < nstages) load_frags(an, t + 1);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < nstages) load_stage(t + 1);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            uint4 b[NS];
#pragma unroll
            for (int h = 0; h < NS; ++h)
                b[h] = *reinterpret_cast<const uint4 *>(buf + (h * kOneRows + wr * 32 + (lane & 31)) * kPPitch +
                                                        (wk * 2 + ks) * 32 + (lane >> 5) * 16);
            mfma_split_sum<NS, true>(a[ks], b, acc, small);
        }
        if (t + 1 < nstages) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int h = 0; h < NS; ++h) a[ks][h] = an[ks][h];
        }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] += small[v];
    __syncthreads();
    float *red = reinterpret_cast<float *>(lds);
    if (wk == 1)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[(wr * 16 + v) * 64 + lane] = acc[v];
    __syncthreads();
    const int64_t i = i0 + wr * 32 + (lane & 31);
    if (wk == 1 || i >= m) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = d_row(v, lane);
        if (c < r) out[(int64_t)c * m + i] = acc[v] + red[(wr * 16 + v) * 64 + lane];
    }
}

// ---------------------------------------------------------------------------------------------
// Q phase of one basis block (r <= 32) and three pieces:  Q_k[j][c] = sum_i delta_k[i][j] P_hat[c][i].
// Wavefront: 128 columns over its own range of rows.  The B operand (N = column, reduction down the
// column) is loaded straight from HBM into the operand layout: lane (x, half) reads the 4 consecutive
// columns j0 + 4 x .. of the rows i0 + 8 half + e, e = 0..7, and column 4 x + q feeds MFMA block q (the
// column blocks are interleaved, which an MFMA does not care about), so one load instruction covers 2
// rows x 512 contiguous bytes.  The 4 wavefronts of a workgroup take consecutive quarters of the
// workgroup's rows and are added in wavefront order at the end; blockIdx.z splits the rows further into
// slabs.
// The two-role kernel below has one workgroup per unit there, 98 KB of LDS, and half of this one's
// requests in flight (8192 x 8192 r = 20 181 us here, 206 there).  With two pieces it has two workgroups
// per unit and takes every rank: 170 us against 178 here, 2048 x 2048 r = 32 21 | 25, 4352 x 7824 r = 6
// three workers 87 | 108.  From two blocks on this kernel needs 326 registers, one wavefront per SIMD.
// ---------------------------------------------------------------------------------------------
constexpr int kQDepth = 2;  // k-steps (16 rows) of delta in flight per wavefront
__global__ __launch_bounds__(kW) void project_q_one_kernel(PtrPack<const float *> deltas,
                                                           const uint4 *__restrict__ afrags,
                                                           PtrPack<float *> outs, int64_t m,
                                                           int64_t n, int r, int64_t ksteps_per_wave,
                                                           int64_t slab_stride) {
    constexpr int NS = 3;
    __shared__ float red[4 * 16 * 64];
    const float *__restrict__ delta = deltas.p[blockIdx.y];
    float *__restrict__ out = outs.p[blockIdx.y] + (int64_t)blockIdx.z * slab_stride;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t jcol = (int64_t)blockIdx.x * 128 + 4 * (lane & 31);
    const bool col_ok = jcol < n;  // n is a multiple of 16: the 4 columns are in or out together
    const int64_t s_begin = ((int64_t)blockIdx.z * 4 + wave) * ksteps_per_wave;
    const int64_t s_end = s_begin + ksteps_per_wave;  // a multiple of kQDepth k-steps

    f32x16_t acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;

    float4 breg[kQDepth][8];
    auto load_kstep = [&](int d, int64_t s) {
        const int64_t ibase = s * 16 + (lane >> 5) * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            breg[d][e] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (ibase + e < m && col_ok) breg[d][e] = stream_load4(delta + (ibase + e) * n + jcol);
        }
    };
#pragma unroll
    for (int d = 0; d < kQDepth; ++d) load_kstep(d, s_begin + d);
    for (int64_t s = s_begin; s < s_end; s += kQDepth) {
#pragma unroll
        for (int d = 0; d < kQDepth; ++d) {
            uint4 a[NS];
#pragma unroll
            for (int h = 0; h < NS; ++h) a[h] = afrags[((s + d) * NS + h) * 64 + lane];
            uint4 b[4][NS];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float4 y = breg[d][e];
                    x[e] = q == 0 ? y.x : q == 1 ? y.y : q == 2 ? y.z : y.w;
                }
                split8<NS>(x, b[q]);
            }
            if (s + d + kQDepth < s_end) load_kstep(d, s + d + kQDepth);
#pragma unroll
            for (int q = 0; q < 4; ++q) mfma_split<NS>(a, b[q], acc[q]);
        }
    }
    // wavefronts 3, 2, 1 hand their sums to wavefront 0, in that order
    for (int w = 3; w >= 1; --w) {
        if (wave == w) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) red[(q * 16 + v) * 64 + lane] = acc[q][v];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[q][v] += red[(q * 16 + v) * 64 + lane];
        }
        __syncthreads();
    }
    if (wave != 0 || !col_ok) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = d_row(v, lane);
        if (c < r) {
#pragma unroll
            for (int q = 0; q < 4; ++q) out[(int64_t)c * n + jcol + q] = acc[q][v];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Reconstruction  delta_hat[i][j] = sum_c P_hat[c][i] Q_bar[c][j]  with fused consumers.
// Workgroup: 32 rows x 256 columns per iteration, swept along j; wavefront w owns the 64 columns
// 64 w .. 64 w + 63 (two 32 x 32 MFMA blocks; A = P_hat fragments with M = i, B = Q_bar fragments
// with N = j).  The accumulators (lane = column, register = row) go through a wavefront-private
// LDS tile so that every access to a matrix element is a 16-byte vector and a wavefront
// instruction covers 4 rows x 256 contiguous bytes, the same shape as a plain streaming kernel:
//   out            : delta_hat is written
//   K > 0          : e_k <- e_k - delta_hat                      (error buffers of Alg. 2)
//   tl_on          : e_k <- (theta - theta_l,k) + e_k            (next pseudo-gradient)
//   apply          : v <- mu v + delta_hat; theta <- theta - lr (delta_hat + mu v)   (OuterOpt)
// ---------------------------------------------------------------------------------------------
constexpr int kRPitch = 64 + 4;  // floats per LDS tile row

template <int NS>
__global__ __launch_bounds__(kW) void reconstruct_mfma_kernel(
    const uint4 *__restrict__ pfrags, const uint4 *__restrict__ qfrags, ReconEpilogue ep,
    int64_t m, int64_t n, int64_t cols_per_wg, int KS) {
    __shared__ __attribute__((aligned(16))) float tile[4][32][kRPitch];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t ib = blockIdx.y;
    const int64_t jbegin = (int64_t)blockIdx.x * cols_per_wg;
    int64_t jend = jbegin + cols_per_wg;
    if (jend > n) jend = n;
    const int64_t nblk = (n + 31) >> 5;
    const int prow = lane >> 4, pc4 = lane & 15;  // epilogue: 4 rows x 16 float4 per instruction

    for (int64_t jt0 = jbegin; jt0 < jend; jt0 += 256) {  // uniform over the workgroup
        const int64_t jt = jt0 + wave * 64;
        f32x16_t d[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) d[nb][v] = 0.f;
        if (jt < jend) {
            const int64_t jb0 = jt >> 5;
            const bool two = jb0 + 1 < nblk;
            for (int s = 0; s < KS; ++s) {
                uint4 a[NS], b0[NS], b1[NS];
#pragma unroll
                for (int h = 0; h < NS; ++h) {
                    a[h] = pfrags[((ib * KS + s) * NS + h) * 64 + lane];
                    b0[h] = qfrags[((jb0 * KS + s) * NS + h) * 64 + lane];
                    b1[h] = two ? qfrags[(((jb0 + 1) * KS + s) * NS + h) * 64 + lane]
                                : make_uint4(0u, 0u, 0u, 0u);
                }
                mfma_split<NS>(a, b0, d[0]);
                mfma_split<NS>(a, b1, d[1]);
            }
        }
        __syncthreads();  // the previous iteration's readers are done with the tile
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                tile[wave][d_row(v, lane)][nb * 32 + (lane & 31)] = d[nb][v];
        __syncthreads();
        const int64_t j = jt + pc4 * 4;
        const bool col_ok = jt < jend && j < n;
        for (int pass = 0; pass < 8; ++pass) {
            const int row = pass * 4 + prow;
            const int64_t i = ib * 32 + row;
            // outside the matrix a lane reads element 0 (dropped) instead of skipping its loads
            // behind a per-lane condition, and stores nothing
            const bool ok = col_ok && i < m;
            const int64_t off = ok ? i * n + j : 0;
            const float4 dv = *reinterpret_cast<const float4 *>(&tile[wave][row][pc4 * 4]);
            if (ep.out) {
                if (ok) stream_store4(ep.out + off, dv);
            }
            float4 tv = make_float4(0.f, 0.f, 0.f, 0.f), vv = tv;
            if (ep.tl_on || ep.apply) tv = stream_load4(ep.theta + off);
            if (ep.apply) vv = stream_load4(ep.vel + off);
            for (int k0 = 0; k0 < ep.K; k0 += 4) {
                float4 x[4], l[4];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    if (k0 + kk < ep.K) {
                        x[kk] = stream_load4(ep.ef.p[k0 + kk] + off);
                        if (ep.tl_on) {
                            if (ep.tl_bf16) {
                                const uint2 bits = stream_load2(
                                    reinterpret_cast<const uint16_t *>(ep.tl.p[k0 + kk]) + off);
                                l[kk] = make_float4(__uint_as_float(bits.x << 16),
                                                    __uint_as_float(bits.x & 0xFFFF0000u),
                                                    __uint_as_float(bits.y << 16),
                                                    __uint_as_float(bits.y & 0xFFFF0000u));
                            } else {
                                l[kk] = stream_load4(
                                    reinterpret_cast<const float *>(ep.tl.p[k0 + kk]) + off);
                            }
                        }
                    }
                }
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    if (k0 + kk < ep.K) {
                        float4 e;
                        e.x = x[kk].x - dv.x; e.y = x[kk].y - dv.y;
                        e.z = x[kk].z - dv.z; e.w = x[kk].w - dv.w;
                        if (ep.tl_on) {
                            e.x = (tv.x - l[kk].x) + e.x; e.y = (tv.y - l[kk].y) + e.y;
                            e.z = (tv.z - l[kk].z) + e.z; e.w = (tv.w - l[kk].w) + e.w;
                        }
                        if (ok) stream_store4(ep.ef.p[k0 + kk] + off, e);
                    }
                }
            }
            if (ep.apply && ok) {
                float4 vn, tn;
                vn.x = fmaf(ep.mu, vv.x, dv.x); vn.y = fmaf(ep.mu, vv.y, dv.y);
                vn.z = fmaf(ep.mu, vv.z, dv.z); vn.w = fmaf(ep.mu, vv.w, dv.w);
                tn.x = fmaf(-ep.lr, fmaf(ep.mu, vn.x, dv.x), tv.x);
                tn.y = fmaf(-ep.lr, fmaf(ep.mu, vn.y, dv.y), tv.y);
                tn.z = fmaf(-ep.lr, fmaf(ep.mu, vn.z, dv.z), tv.z);
                tn.w = fmaf(-ep.lr, fmaf(ep.mu, vn.w, dv.w), tv.w);
                stream_store4(ep.vel + off, vn);
                stream_store4(ep.theta + off, tn);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The whole pass between two compressions, fused with the P phase of the next one (outer step
// t >= 2), for up to KC workers:
//   d        = P_hat_prev Q_bar_prev^T             (tile by tile, never written)
//   e_k      = delta_k - d ;  delta_k = (theta - theta_l,k) + e_k     -> stored over delta_k
//   P_k     += delta_k Q_in                        (accumulated while the tile is on chip)
//   apply    : v <- mu v + d ; theta <- theta - lr (d + mu v)
// Same tiling as the reconstruction kernel (32 rows x 256 columns per iteration, wavefront w owns
// 64 columns).  After the elementwise step the new delta_k tile is written to LDS as bf16 pieces
// in the layout of the P-phase kernel (row-major, reduction index contiguous) and multiplied with
// the basis fragments of its 64 columns: delta is read from HBM once for all of this.  A
// workgroup leaves the partial P_k of its rows and column range in slab blockIdx.x; the slabs of
// a row block are added afterwards in slab order.
// ---------------------------------------------------------------------------------------------
// LDS written by some lanes of a wavefront and read by others: the data share unit executes one
// wavefront's instructions in order, so only the compiler has to be kept from reordering.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of one wavefront's tile: fp32, or bf16 pieces
constexpr int round_tile_bytes(int ns) {
    return 32 * kRPitch * 4 > ns * 32 * kPPitch ? 32 * kRPitch * 4 : ns * 32 * kPPitch;
}

template <int NS, int CB, int KC, bool TLBF16>
__global__ __launch_bounds__(kW) void round_mfma_kernel(
    const uint4 *__restrict__ pfrags, const uint4 *__restrict__ qfrags, int KS,
    const uint4 *__restrict__ bfrags, ReconEpilogue ep, PtrPack<float *> pslab, int64_t m,
    int64_t n, int r, int tiles, int64_t slab_stride) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // Per wavefront: the fp32 staging tile of d and the bf16 pieces of its delta tile, which are never
    // in use together (round_tile_bytes), and the basis fragments of its 64 columns.  With three
    // pieces and two basis blocks that is 151 KB of the compute unit's 160.  (Fragments read from L2
    // inside the loop wait for every HBM request made before them: 338 us against 312 for 5008 x
    // 3376 at r = 56 with three fp32 workers.)
    constexpr int kTileBytes = round_tile_bytes(NS);
    constexpr int kBasisBytes = 4 * CB * NS * 1024;
    unsigned char *btile = smem + (threadIdx.x >> 6) * kTileBytes;
    float *tile = reinterpret_cast<float *>(btile);
    uint4 *basis_lds = reinterpret_cast<uint4 *>(smem + 4 * kTileBytes + (threadIdx.x >> 6) * kBasisBytes);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t ib = blockIdx.y;
    // 256-column tiles of the row block, dealt evenly to its workgroups, the longer ranges first
    const uint32_t chunks = gridDim.x, end_at = (blockIdx.x + 1) * (uint32_t)tiles + chunks - 1;
    const int64_t jbegin = (int64_t)((end_at - (uint32_t)tiles) / chunks) * 256;
    int64_t jend = (int64_t)(end_at / chunks) * 256;
    if (jend > n) jend = n;
    const int64_t nblk = (n + 31) >> 5;
    const int prow = lane >> 4, pc4 = lane & 15;
    const int64_t row0 = ib * 32 + prow;  // pass p covers row row0 + 4 p
    typedef typename std::conditional<TLBF16, uint2, float4>::type traw_t;

    f32x16_t acc[KC][CB];
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[k][cb][v] = 0.f;

    // operands of the item (column tile, worker) in flight
    float4 x[8], tv[8], vv[8];
    traw_t lraw[8];
    auto issue = [&](int64_t jt, int k, bool with_theta, bool with_vel) {
        const int64_t j = jt + pc4 * 4;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            // outside the matrix: element 0 instead (what comes back is never used: the new
            // delta is forced to zero there and nothing is stored), so that no lane branches
            const bool okp = j < n && row0 + 4 * p < m;
            const int64_t off = okp ? (row0 + 4 * p) * n + j : 0;
            x[p] = stream_load4(ep.ef.p[k] + off);
            if constexpr (TLBF16)
                lraw[p] = stream_load2(reinterpret_cast<const uint16_t *>(ep.tl.p[k]) + off);
            else
                lraw[p] = stream_load4(reinterpret_cast<const float *>(ep.tl.p[k]) + off);
            if (with_theta) tv[p] = stream_load4(ep.theta + off);
            if (with_vel) vv[p] = stream_load4(ep.vel + off);
        }
    };
    const int Kw = ep.K;
    // This wavefront's tiles are the columns jw + 256 t, t = 0 .. nw - 1.  They are visited in
    // rotated order: the workgroups of a launch start together, and without the rotation all
    // of them would sweep the same columns of different rows at the same time, rows whose
    // distance in memory is the same multiple of a power of two for the common matrix widths.
    const int64_t jw = jbegin + wave * 64;
    const int64_t nw = jw < jend ? (jend - jw + 255) >> 8 : 0;
    // Starting tile: groups of 8 consecutive row blocks start a quarter of the range apart
    // (4 starting points).  Measured against a start of ib mod nw (every row block its own):
    // 5 - 6 % faster on the 8192-column shapes, no difference at 28672 columns; with 8 or 16
    // starting points, or groups of 1 or 2 row blocks, the gain is smaller or gone.
    const int64_t pp = nw < 4 ? nw : 4;
    const int64_t shift = nw > 0 ? ((ib >> 3) % pp) * nw / pp : 0;
    auto tile_at = [&](int64_t i) {
        const int64_t t = i + shift;
        return jw + ((t >= nw ? t - nw : t) << 8);
    };
    if (nw > 0) issue(tile_at(0), 0, true, ep.apply && Kw == 1);
    for (int64_t it = 0; it < nw; ++it) {
        const int64_t jt = tile_at(it);
        // ---- d = P_hat_prev Q_bar_prev^T for this wavefront's 32 x 64 tile
        f32x16_t d[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) d[nb][v] = 0.f;
        {
            const int64_t jb0 = jt >> 5;
            const bool two = jb0 + 1 < nblk;
            for (int s = 0; s < KS; ++s) {
                uint4 a[NS], b0[NS], b1[NS];
#pragma unroll
                for (int h = 0; h < NS; ++h) {
                    a[h] = pfrags[((ib * KS + s) * NS + h) * 64 + lane];
                    b0[h] = qfrags[((jb0 * KS + s) * NS + h) * 64 + lane];
                    b1[h] = two ? qfrags[(((jb0 + 1) * KS + s) * NS + h) * 64 + lane]
                                : make_uint4(0u, 0u, 0u, 0u);
                }
                mfma_split<NS>(a, b0, d[0]);
                mfma_split<NS>(a, b1, d[1]);
            }
        }
        wave_lds_sync();  // earlier readers of the staging tile and of the basis are done
        // this tile's basis fragments: 4 k-steps x CB blocks x NS pieces
#pragma unroll
        for (int f = 0; f < 4 * CB * NS; ++f)
            basis_lds[f * 64 + lane] = bfrags[((jt >> 4) * CB * NS + f) * 64 + lane];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                tile[d_row(v, lane) * kRPitch + nb * 32 + (lane & 31)] = d[nb][v];
        wave_lds_sync();
        float4 dv[8];
#pragma unroll
        for (int p = 0; p < 8; ++p)
            dv[p] = *reinterpret_cast<const float4 *>(&tile[(p * 4 + prow) * kRPitch + pc4 * 4]);
        const int64_t j = jt + pc4 * 4;
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            if (k < Kw) {
                const bool last = k == Kw - 1;
                float *__restrict__ e = ep.ef.p[k];
                wave_lds_sync();  // the previous item's fragments have been read
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const bool okp = j < n && row0 + 4 * p < m;
                    const int64_t off = (row0 + 4 * p) * n + j;
                    float4 l;
                    if (TLBF16) {
                        const uint2 bits = *reinterpret_cast<const uint2 *>(&lraw[p]);
                        l = make_float4(__uint_as_float(bits.x << 16),
                                        __uint_as_float(bits.x & 0xFFFF0000u),
                                        __uint_as_float(bits.y << 16),
                                        __uint_as_float(bits.y & 0xFFFF0000u));
                    } else {
                        l = *reinterpret_cast<const float4 *>(&lraw[p]);
                    }
                    float4 g;
                    g.x = (tv[p].x - l.x) + (x[p].x - dv[p].x);
                    g.y = (tv[p].y - l.y) + (x[p].y - dv[p].y);
                    g.z = (tv[p].z - l.z) + (x[p].z - dv[p].z);
                    g.w = (tv[p].w - l.w) + (x[p].w - dv[p].w);
                    if (okp) {
                        stream_store4(e + off, g);
                    } else {
                        g = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                    uint32_t lo[NS], hi[NS];
                    split2<NS>(g.x, g.y, lo);
                    split2<NS>(g.z, g.w, hi);
#pragma unroll
                    for (int h = 0; h < NS; ++h)
                        *reinterpret_cast<uint2 *>(btile + (h * 32 + p * 4 + prow) * kPPitch +
                                                   pc4 * 8) = make_uint2(lo[h], hi[h]);
                    if (last && ep.apply && okp) {
                        float4 vn, tn;
                        vn.x = fmaf(ep.mu, vv[p].x, dv[p].x); vn.y = fmaf(ep.mu, vv[p].y, dv[p].y);
                        vn.z = fmaf(ep.mu, vv[p].z, dv[p].z); vn.w = fmaf(ep.mu, vv[p].w, dv[p].w);
                        tn.x = fmaf(-ep.lr, fmaf(ep.mu, vn.x, dv[p].x), tv[p].x);
                        tn.y = fmaf(-ep.lr, fmaf(ep.mu, vn.y, dv[p].y), tv[p].y);
                        tn.z = fmaf(-ep.lr, fmaf(ep.mu, vn.z, dv[p].z), tv[p].z);
                        tn.w = fmaf(-ep.lr, fmaf(ep.mu, vn.w, dv[p].w), tv[p].w);
                        stream_store4(ep.vel + off, vn);
                        stream_store4(ep.theta + off, tn);
                    }
                }
                // operands of the next item, in flight while this one is multiplied
                if (!last) {
                    issue(jt, k + 1, false, ep.apply && k + 1 == Kw - 1);
                } else if (it + 1 < nw) {
                    issue(tile_at(it + 1), 0, true, ep.apply && Kw == 1);
                }
                wave_lds_sync();
                // NS == 3, or one basis block: the tile's products of a block in an accumulator of their
                // own, added to the sum once (mfma_split_sum: the fp32 error of a long sum is the
                // rounding of its large terms).  Block by block: for all of them at once the registers
                // do not last.
                auto load_b = [&](int s, uint4 (&b)[NS]) {
#pragma unroll
                    for (int h = 0; h < NS; ++h)
                        b[h] = *reinterpret_cast<const uint4 *>(
                            btile + (h * 32 + (lane & 31)) * kPPitch + s * 32 + (lane >> 5) * 16);
                };
                auto product = [&](int cb, int s, const uint4 (&b)[NS], f32x16_t &sum) {
                    uint4 a[NS];
#pragma unroll
                    for (int h = 0; h < NS; ++h)
                        a[h] = basis_lds[((s * CB + cb) * NS + h) * 64 + lane];
                    mfma_split<NS>(a, b, sum);
                };
                if constexpr (NS == 3 || CB == 1) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        f32x16_t part;
#pragma unroll
                        for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            uint4 b[NS];
                            load_b(s, b);
                            product(cb, s, b, part);
                        }
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[k][cb][v] += part[v];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        uint4 b[NS];
                        load_b(s, b);
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) product(cb, s, b, acc[k][cb]);
                    }
                }
            }
        }
    }
    // add the four wavefronts' partial P_k (wavefronts 3, 2, 1 hand over to 0, in that order)
    __syncthreads();
    float *red = reinterpret_cast<float *>(smem);
    for (int w = 3; w >= 1; --w) {
        if (wave == w) {
#pragma unroll
            for (int k = 0; k < KC; ++k)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        red[((k * CB + cb) * 16 + v) * 64 + lane] = acc[k][cb][v];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int k = 0; k < KC; ++k)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[k][cb][v] += red[((k * CB + cb) * 16 + v) * 64 + lane];
        }
        __syncthreads();
    }
    if (wave != 0) return;
    const int64_t i = ib * 32 + (lane & 31);
    if (i >= m) return;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        if (k < Kw) {
            float *__restrict__ out = pslab.p[k] + (int64_t)blockIdx.x * slab_stride;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int c = cb * 32 + d_row(v, lane);
                    if (c < r) out[(int64_t)c * m + i] = acc[k][cb][v];
                }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Q phase in the two-role form of project_p_ws_kernel, for any number of basis blocks (one: with two
// pieces only).  A workgroup owns
// 128 columns and a range of rows, swept in stages of 64 rows (4 k-steps).  Producer thread
// (column quad c4, row group rg) requests 8 rows x 4 columns per stage -- one instruction of a
// wavefront covers 2 rows x 512 bytes -- and holds, for each of its 4 columns, exactly the 8
// reduction-consecutive values one lane feeds to the matrix cores: it splits them into bf16
// pieces and writes them to LDS in operand order, so that a consumer fetches one 16 x 32 operand
// block of one piece as 1 KB of consecutive LDS.  The consumers form a WCB x (4 / WCB) grid:
// wavefront w owns the CBW basis blocks of group w % WCB and WCB of the four 32-column blocks.
// Register sets, buffers, barriers and clamping as in the P kernel.
// ---------------------------------------------------------------------------------------------
// LONE: at most one workgroup per compute unit, which then has twice the registers: always with three
// pieces (98 KB of LDS), with two where the plan says so.  Accumulators of the small products as in the P
// kernel, LONE at 4 basis blocks too; accumulators that take the k-steps in turn: four for one block, LONE
// two.  Error against fp64 of two pieces, 8192 x 8064 four workers: r = 64 5.9e-7 (one chain: 7.2e-7), r =
// 100 7.0e-7 (one chain with all products in it: 1.06e-6); of three, 3056 x 6336 five workers r = 48 1.5e-7
// (one chain: 2.9e-7); no difference in time.
template <int NS, int BLOCKS, bool LONE>
constexpr bool kApartQ = NS >= 2 && BLOCKS <= (LONE ? 4 : 2);
template <int NS, int BLOCKS, bool LONE>
constexpr int kChainsQ = NS < 2 ? 1 : BLOCKS == 1 ? 4 : LONE && BLOCKS <= 4 ? 2 : 1;
template <int NS, int CBW, int WCB, bool LONE = NS == 3>
__global__ __launch_bounds__(kWs, NS == 2 && CBW * WCB == 1 ? 4 : 1) void project_q_ws_kernel(PtrPack<const float *> deltas,
                                                           const uint4 *__restrict__ afrags,
                                                           PtrPack<float *> outs, int64_t m,
                                                           int64_t n, int r, int64_t ksteps_per_wg,
                                                           int64_t slab_stride,
                                                           uint32_t *__restrict__ amax_record,
                                                           const float *__restrict__ out_scale,
                                                           const uint32_t *__restrict__ guard) {
    constexpr int CB = WCB * CBW;
    constexpr int QW = WCB;               // column blocks per consumer: 4 / (4 / WCB)
    constexpr int kBuf = 16 * NS * 1024;  // 4 k-steps x 4 column blocks x NS pieces x 1 KB
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    if (guard != nullptr && f16_range_ok(*guard)) return;  // uniform over the launch
    const float *__restrict__ delta = deltas.p[blockIdx.y];
    float *__restrict__ out = outs.p[blockIdx.y] + (int64_t)blockIdx.z * slab_stride;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t j0 = (int64_t)blockIdx.x * 128;
    const int64_t s_begin = (int64_t)blockIdx.z * ksteps_per_wg;  // a multiple of 4
    const int64_t nstages = ksteps_per_wg >> 2;

    if (wave >= 4) {  // ---------------------------------------------------------- producers
        const int tid = threadIdx.x - kW;
        const int c4 = tid & 31, rg = tid >> 5;
        const bool col_ok = j0 + c4 * 4 < n;
        float amax = 0.f;  // NS == 1: largest |delta| this thread has laid down
        auto load_stage = [&](float4 (&set)[8], int64_t t) {
            const int64_t tc = t < nstages ? t : nstages - 1;
            const int64_t i0 = (s_begin + 4 * tc) * 16 + rg * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool ok = col_ok && i0 + e < m;
                set[e] = stream_load4(ok ? delta + (i0 + e) * n + j0 + c4 * 4 : delta);
            }
        };
        auto store_stage = [&](const float4 (&set)[8], unsigned char *buf, int64_t t) {
            const int64_t i0 = (s_begin + 4 * t) * 16 + rg * 8;
            float v[4][8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool ok = col_ok && i0 + e < m;
                v[0][e] = ok ? set[e].x : 0.f;
                v[1][e] = ok ? set[e].y : 0.f;
                v[2][e] = ok ? set[e].z : 0.f;
                v[3][e] = ok ? set[e].w : 0.f;
            }
            if constexpr (NS == 1) {
                constexpr float kUp = (float)(1 << kF16DeltaShift);
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        amax = fmaxf(amax, fabsf(v[x][e]));
                        v[x][e] *= kUp;
                    }
            }
            // operand block (k-step rg / 2, column block c4 / 8), lane (rg % 2) 32 + column
            // (the two low bits of the lane slot are swizzled so that the 16 lanes of one LDS
            // pass, which differ in c4, fall on 16 different bank groups; a consumer reads the
            // 64 slots of a block in the same permutation)
            unsigned char *blk = buf + ((rg >> 1) * 4 + (c4 >> 3)) * NS * 1024 +
                                 ((rg & 1) * 32 + (c4 & 7) * 4) * 16;
            const int sw = (((c4 >> 2) & 1) << 1) | ((c4 >> 3) & 1);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                uint4 pieces[NS];
                split8<NS>(v[x], pieces);
#pragma unroll
                for (int h = 0; h < NS; ++h)
                    *reinterpret_cast<uint4 *>(blk + h * 1024 + (x ^ sw) * 16) = pieces[h];
            }
        };
        auto step = [&](float4 (&set)[8], int64_t stage, bool refill) {
            store_stage(set, lds + (stage & 1) * kBuf, stage);
            if (refill) load_stage(set, stage + 2);
            lds_barrier();
            __builtin_amdgcn_sched_barrier(0);
        };
        float4 set0[8], set1[8];
        load_stage(set0, 0);
        load_stage(set1, 1);
        step(set0, 0, true);
        int64_t t = 0;
        for (; t + 1 < nstages; t += 2) {
            step(set1, t + 1, true);
            step(set0, t + 2, true);
        }
        if (t < nstages) step(set1, t + 1, false);
        if constexpr (NS == 1) record_amax(amax, amax_record);
        return;
    }
    // -------------------------------------------------------------------------------- consumers
    const int wcb = wave % WCB, wq = wave / WCB;
    constexpr bool kApart = kApartQ<NS, CBW * QW, LONE>;
    constexpr int kTurns = kChainsQ<NS, CBW * QW, LONE>;
    f32x16_t acc[kTurns][CBW][QW], small[kApart ? CBW : 1][kApart ? QW : 1];
#pragma unroll
    for (int a = 0; a < CBW; ++a)
#pragma unroll
        for (int b = 0; b < QW; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
#pragma unroll
                for (int t = 0; t < kTurns; ++t) acc[t][a][b][v] = 0.f;
                if constexpr (kApart) small[a][b][v] = 0.f;
            }
    constexpr int AD = CBW * NS <= 2 ? 4 : 2;  // as in project_p_ws_kernel
    uint4 a[AD][CBW][NS];                      // fragments of k-step g in ring position g % AD
    const int64_t gmax = s_begin + ksteps_per_wg - 1;
    auto load_frags = [&](int64_t g, int pos) {
        const int64_t gc = g < gmax ? g : gmax;
#pragma unroll
        for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
            for (int h = 0; h < NS; ++h)
                a[pos][cb][h] = afrags[((gc * CB + wcb * CBW + cb) * NS + h) * 64 + lane];
    };
#pragma unroll
    for (int g = 0; g < AD; ++g) load_frags(s_begin + g, g);
    lds_barrier();
    for (int64_t t = 0; t < nstages; ++t) {
        const unsigned char *buf = lds + (t & 1) * kBuf;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            uint4 b[QW][NS];
#pragma unroll
            for (int q = 0; q < QW; ++q)
#pragma unroll
                for (int h = 0; h < NS; ++h)
                    b[q][h] = *reinterpret_cast<const uint4 *>(
                        buf + ((ks * 4 + wq * QW + q) * NS + h) * 1024 +
                        (lane ^ ((((lane >> 4) & 1) << 1) | ((wq * QW + q) & 1))) * 16);
#pragma unroll
            for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
                for (int q = 0; q < QW; ++q)
                    mfma_split_sum<NS, kApart>(a[ks % AD][cb], b[q], acc[ks % kTurns][cb][q],
                                               small[kApart ? cb : 0][kApart ? q : 0]);
            load_frags(s_begin + t * 4 + ks + AD, ks % AD);
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier();
    }
#pragma unroll
    for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
        for (int q = 0; q < QW; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if constexpr (kApart) acc[0][cb][q][v] += small[cb][q][v];
                if constexpr (kTurns >= 2) acc[0][cb][q][v] += acc[1][cb][q][v];
                if constexpr (kTurns == 4) acc[0][cb][q][v] += acc[2][cb][q][v] + acc[3][cb][q][v];
            }
#pragma unroll
    for (int q = 0; q < QW; ++q) {
        const int64_t j = j0 + (wq * QW + q) * 32 + (lane & 31);
        if (j >= n) continue;
#pragma unroll
        for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int c = (wcb * CBW + cb) * 32 + d_row(v, lane);
                if (c < r) out[(int64_t)c * n + j] = NS == 1 ? acc[0][cb][q][v] * out_scale[c] : acc[0][cb][q][v];
            }
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static inline int ns_of(int mma) { return mma == DLCX_MMA_F32 ? 3 : 2; }
static inline int cb_of(int r) { return r <= 32 ? 1 : r <= 64 ? 2 : r <= 128 ? 4 : 8; }
static inline size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

struct QPlan {
    int S;
    int64_t ksteps_per_wave, KS;
    bool lone;  // at most one workgroup per compute unit, the kernel's form for that
};

// Splits of the reduction.  A projection has one workgroup per 128 rows (P; 64 in one case, p_plan) or
// columns (Q) of the output and worker; where that leaves compute units without one, the reduction is
// split and the partial sums, one slab per split and worker, are added afterwards (sum_partials).
constexpr int64_t kQUnits = 256;  // compute units
constexpr int64_t kPShort = 1024;  // columns up to which the P kernel may take 64 rows
// Most splits a plan may choose for `wgs` workgroups per split, whatever the reduction's length and
// the rank: no more than two workgroups per compute unit.
static int64_t most_splits(int64_t wgs) {
    const int64_t s = ceil_div(2 * kQUnits, wgs);
    return s > 64 ? 64 : s;
}
static int64_t out_wgs(int64_t side) { return ceil_div(side, 128); }
// Most splits of a reduction by its length: two stages of 64 columns (P), two pipeline rounds of every
// wavefront (Q: 2 x 4 x 2 k-steps of 16 rows) each.
static int64_t most_p_splits(int64_t n) { return ceil_div(ceil_div(n, 64), 2); }
static int64_t most_q_splits(int64_t m) { return ceil_div(m, 256); }
// Slabs a workspace for K workers has room for: enough for any smaller number of workers and any
// smaller rank that is later run in it.
static int64_t slab_room(int64_t side, int K, int64_t by_length) {
    int64_t room = 0;
    for (int k = 1; k <= K; ++k) {
        int64_t s = most_splits(out_wgs(side) * k);
        if (s > by_length) s = by_length;
        if (s > 1 && s * k > room) room = s * k;
    }
    return room;
}

// The cheapest number of splits, smin to smax, of a reduction over `length`: rounds of the launch x
// length of a workgroup's share in whole `granule`s (and 128 more to start and drain), plus the slabs,
// written and read, in the same unit (512 bytes of delta on one compute unit).  Two workgroups on some
// units and one on the others is as slow as two everywhere.  Measured (us, chosen | two per unit, the
// rule before): Q of 8192 x 1024 r = 64 8 splits 39 | 16: 47; 2048 x 2048 r = 32 4: 21 | 8: 28; r = 64
// 4: 26 | 8: 33; 8192 x 3008 r = 32 5: 74 | 6: 101; 4096 x 4096 r = 64 2: 59 | 4: 68; 5008 x 3376 r = 56
// three workers, three pieces 3: 66 | 7: 90.  P, 64 rows and no splits before: 2048 x 8192 r = 32 55 |
// 125, r = 100 88 | 163; 2048 x 2048 r = 64 26 | 41; 3008 x 5008 r = 100 two workers 54 | 107; 256 x 8192
// r = 16 one worker 21 | 102; 1120 x 6688 r = 210 one worker 34 | 170.
static int64_t split_cost(int64_t wgs, int64_t length, int64_t granule, int64_t slab_elements, int64_t s) {
    const int64_t share = ceil_div(ceil_div(length, s), granule) * granule;
    return ceil_div(wgs * s, kQUnits) * (share + 128) + s * slab_elements / 16384;
}
static int64_t best_splits(int64_t wgs, int64_t length, int64_t granule, int64_t slab_elements,
                           int64_t smin, int64_t smax) {
    int64_t S = smin;
    for (int64_t s = smin + 1; s <= smax; ++s)
        if (split_cost(wgs, length, granule, slab_elements, s) < split_cost(wgs, length, granule, slab_elements, S))
            S = s;
    return S;
}

struct PPlan {
    int rows;        // rows of delta per workgroup
    int S;           // column splits
    int64_t stages;  // stages of 64 columns of a split
    bool one_role;   // project_p_one_kernel
    bool lone;       // at most one workgroup per compute unit
};
// 64 rows per workgroup where the matrix cores set the pace (4 or 8 basis blocks), the rows then still
// fit the units in one round and the reduction is short: a longer chain of stages is not what such a
// launch waits for.  64 | 128 rows, us: 8192 x 512 r = 100 two workers 21 | 27, 2176 x 256 r = 145 16 |
// 20, 7136 x 640 r = 74 22 | 25, 6000 x 1024 r = 100 21 | 23; 3008 x 2048 r = 200 41 | 39, 2048 x 3072 r =
// 200 three pieces 81 | 76.
// One basis block and a workgroup for nearly every unit: the one-role kernel, unless the reduction is long
// and 128 rows deal evenly (one for every unit, or nearly two).  one-role | two-role, us, r = 20, two
// workers, two pieces: 14336 x 512 18.3 | 18.3; 15360 x 512 18.4 | 19.2, x 2048 54.0 | 55.8; 16384 x 512
// 18.9 | 20.5, x 4096 126 | 131, x 8192 221 | 216; 16896 x 512 21.7 | 27.2, x 4096 129 | 165, x 8192 250 |
// 279; 24576 x 4096 152 | 185, x 8192 315 | 344; 32768 x 1024 64 | 71, x 4096 213 | 234, x 8192 411 | 350;
// 65536 x 1024 117 | 132, x 4096 410 | 428, x 8192 791 | 699.  Three pieces: 16384 x 1024 36.5 | 40.3, x
// 8192 221 | 210; 16896 x 8192 340 | 374; 32768 x 1024 67 | 76, x 4096 244 | 261, x 8192 459 | 420; 7232 x
// 704 r = 6 four workers 23.5 | 25.0.  Errors against 64 bits are within 2 %.
constexpr int64_t kPLong = 4096;
constexpr int64_t kPOneFrom = 224;  // workgroups of 128 rows
static PPlan p_plan(int64_t m, int64_t n, int r, int K) {
    PPlan p;
    const int64_t stages = ceil_div(n, 64);
    p.rows = cb_of(r) >= 4 && n <= kPShort && ceil_div(m, 64) * K <= kQUnits ? 64 : 128;
    const int64_t wgs = ceil_div(m, p.rows) * K;
    p.one_role = cb_of(r) == 1 && wgs >= kPOneFrom && !(n > kPLong && (wgs <= kQUnits || 2 * wgs > 3 * kQUnits));
    int64_t smax = most_splits(wgs), S = 1;
    if (smax > most_p_splits(n)) smax = most_p_splits(n);
    // (a second workgroup on every unit does not pay here: 8192 x 8192 r = 64 271 us split in two, 240 not)
    // (where a workgroup has little to stream the slabs cost two and a half times the estimate's: 3264 x 320
    // r = 246 two workers 22.8 us split in two, 19.3 not, 8192 x 256 r = 200 21.5 | 17.7)
    const int64_t slab = (int64_t)K * r * m * (n <= kPShort ? 5 : 2) / 2;
    if (wgs < kQUnits && !p.one_role) S = best_splits(wgs, n, 64, slab, 1, smax);
    p.stages = ceil_div(stages, S);
    p.S = (int)ceil_div(stages, p.stages);
    p.lone = wgs * p.S <= kQUnits;
    return p;
}

static QPlan q_plan(int ns, bool f16, int64_t m, int64_t n, int r, int K) {
    QPlan p;
    const int cb = cb_of(r);
    p.lone = ns == 3;
    const int64_t wgs = out_wgs(n) * K;
    int64_t smax = most_splits(wgs);
    if (smax > most_q_splits(m)) smax = most_q_splits(m);
    int64_t S = 1;
    if (ns == 3 && cb == 1) {
        // the one-role kernel: two workgroups for every unit, whatever remains.  (Fewer splits, with
        // longer fp32 sums, are up to 1.7 times as far from fp64: 6112 x 6864 r = 4.)
        S = smax;
    } else if (wgs >= kQUnits) {
        // every compute unit has a workgroup: two, except at 8 basis blocks, where one fills it
        if (cb < 8) S = smax;
    } else if (!f16 && (ns == 2 || cb == 8)) {
        // Sums no less accurate than those of one accumulator for all piece products in s0 splits, two
        // workgroups for every unit (one at 8 basis blocks), whatever remains: the squared error goes with
        // the roundings of a sum over its splits, and again over the splits.  Where one accumulator takes
        // them all (4, 8 blocks) that needs s0 splits, apart from the small products (2 blocks) s0 / sqrt(3),
        // in two accumulators as well (lone) s0 / sqrt(12); one block has four for a workgroup, where the
        // one-role kernel had one for each of four wavefronts: 0.45 s0 by measurement.
        const int64_t full = ceil_div(cb == 8 ? kQUnits : 2 * kQUnits, wgs), s0 = full < smax ? full : smax;
        const int64_t slab = (int64_t)K * r * n, granule = 64 * kQDepth;
        S = best_splits(wgs, m, granule, slab, cb == 1 ? ceil_div(s0 * 45, 100) : cb == 2 ? ceil_div(s0 * 58, 100) : s0, smax);
        const int64_t fit = kQUnits / wgs < smax ? kQUnits / wgs : smax, least = ceil_div(s0 * 29, 100);
        if (ns == 2 && (cb == 2 || cb == 4) && least <= fit) {
            const int64_t one = best_splits(wgs, m, granule, slab, least, fit);
            // (at 4 blocks one workgroup streams 4 - 8 % slower than two: 8192 x 8192 r = 128 two workers
            // 142 us in two splits, 137 in four; 4096 x 4096 four workers 78 and 83)
            p.lone = split_cost(wgs, m, granule, slab, one) * 10 <=
                     split_cost(wgs, m, granule, slab, S) * (cb == 4 ? 9 : 10);
            if (p.lone) S = one;
        }
    } else {
        S = best_splits(wgs, m, 64 * kQDepth, (int64_t)K * r * n, 1, smax);
    }
    const int64_t kpw = ceil_div(ceil_div(m, 16), S * 4);
    p.ksteps_per_wave = ceil_div(kpw, kQDepth) * kQDepth;
    p.S = (int)ceil_div(ceil_div(m, 16), p.ksteps_per_wave * 4);  // none without rows
    p.KS = p.ksteps_per_wave * 4 * p.S;
    return p;
}

// scratch of the fp16 form at the end of the fragment area: in_scale[256], out_scale[256], record
constexpr size_t kF16ScratchBytes = (2 * DLCX_MAX_RANK + 64) * sizeof(float);

size_t mfma_project_workspace_bytes(int mma, int64_t m, int64_t n, int r, int K) {
    // DLCX_MMA_F16: one fp16 piece beside the two bf16 pieces of the stand-by launch
    const int ns = mma == DLCX_MMA_F16 ? 3 : ns_of(mma), cb = cb_of(r);
    const size_t p_frags = (size_t)ceil_div(n, 64) * 4 * cb * ns * 1024;
    // k-steps are rounded up to kQDepth per wavefront: 8 more for every split (most of them with one
    // worker, if the workspace is later used for fewer workers)
    int64_t splits = most_splits(out_wgs(n));
    if (splits > most_q_splits(m)) splits = most_q_splits(m);
    const size_t q_frags = (size_t)(ceil_div(m, 16) + 8 * splits) * cb * ns * 1024;
    const size_t slabs = (size_t)slab_room(n, K, most_q_splits(m)) * r * n * sizeof(float);
    const size_t p_slabs = (size_t)slab_room(m, K, most_p_splits(n)) * r * m * sizeof(float);
    const size_t a = a256(p_frags) + a256(p_slabs), b = a256(q_frags) + a256(slabs);
    return (a > b ? a : b) + (mma == DLCX_MMA_F16 ? a256(kF16ScratchBytes) : 0);
}

template <int NS>
static int pack_kcontig(const KContig &p, hipStream_t st) {
    Timed timed(KID_PACK, st);
    hipLaunchKernelGGL(pack_kcontig_kernel<NS>, dim3((unsigned)ceil_div(p.count(), 4)), dim3(kW), 0, st, p);
    return check_launch("pack_kcontig");
}

template <int NS>
static int pack_sweep(const KContig &basis, const KStrided &p_hat, const KStrided &q_bar,
                      hipStream_t st) {
    const int64_t nf = basis.count() + p_hat.count() + q_bar.count();
    Timed timed(KID_PACK, st);
    hipLaunchKernelGGL(pack_sweep_kernel<NS>, dim3((unsigned)ceil_div(nf, 4)), dim3(kW), 0, st, basis,
                       p_hat, q_bar);
    return check_launch("pack_sweep");
}

// scales and record of the fp16 form inside its scratch block
struct F16Scratch {
    float *in_scale, *out_scale;
    uint32_t *record;
};
static F16Scratch f16_scratch(void *block) {
    F16Scratch f;
    f.in_scale = reinterpret_cast<float *>(block);
    f.out_scale = f.in_scale + DLCX_MAX_RANK;
    f.record = reinterpret_cast<uint32_t *>(f.out_scale + DLCX_MAX_RANK);
    return f;
}
// the scales of the fp16 form, then both forms of the fragments
static int pack_f16(const KContig &p, uint4 *frags_f16, const F16Scratch &f, hipStream_t st) {
    Timed timed(KID_PACK, st);
    hipLaunchKernelGGL(basis_scale_kernel, dim3((unsigned)p.nrows), dim3(kW), 0, st, p.src, p.L,
                       f.in_scale, f.out_scale, f.record);
    int rc = check_launch("basis_scale");
    if (rc != DLCX_OK) return rc;
    hipLaunchKernelGGL(pack_f16_kernel, dim3((unsigned)ceil_div(p.count(), 4)), dim3(kW), 0, st, p,
                       frags_f16, f.in_scale);
    return check_launch("pack_f16");
}

template <int NS, int CBW, int WC, int WR, int RB = 4, bool LONE = NS == 3, int kSets = 2>
static int project_p_ws_launch(const PPlan &pl, const PtrPack<const float *> &delta,
                               const uint4 *frags, const PtrPack<float *> &out, int64_t m,
                               int64_t n, int r, int K, hipStream_t st, uint32_t *record = nullptr,
                               const float *out_scale = nullptr, const uint32_t *guard = nullptr) {
    constexpr int lds = 2 * NS * 32 * RB * kPPitch;
    static size_t granted = 0;
    int rc = grant_dynamic_lds(
        reinterpret_cast<const void *>(project_p_ws_kernel<NS, CBW, WC, WR, RB, LONE, kSets>), lds,
        &granted, "project_p attribute");
    if (rc != DLCX_OK) return rc;
    const dim3 grid((unsigned)ceil_div(m, 32 * RB), (unsigned)K, (unsigned)pl.S);
    hipLaunchKernelGGL((project_p_ws_kernel<NS, CBW, WC, WR, RB, LONE, kSets>), grid, dim3(kWs), lds, st,
                       delta, frags, out, m, n, r, pl.stages, (int64_t)r * m, record, out_scale,
                       guard);
    return DLCX_OK;
}

// Columns from which the producers of the fp16 P kernel hold three register sets, stages requested ahead, where a
// workgroup has a unit to itself (8 basis blocks; two sets are 64 KB in flight there).  r = 256 four workers, us
// with two sets | three: 8192 x 1024 67 | 67, x 2048 94 | 93, x 4096 152 | 150, x 5120 163 | 162, x 6144 208 | 208,
// x 8192 231 | 223, x 12288 339 | 327, x 16384 438 | 426, x 20480 558 | 532, x 28672 764 | 732; r = 190 8192 x
// 8192 238 | 239, x 28672 731 | 710, 28672 x 8192 826 | 811.  At 4 blocks it gained nothing (8192 x 4096 r = 100
// 147 | 145, 8192 x 8192 r = 66 195 | 194).
constexpr int64_t kPDeep = 8192;

// The projection at 4 or 8 basis blocks (ranks above 64) in its fp16 form, where the matrix cores
// and not the stream of delta set the pace: one fp16 product per block instead of three bf16
// ones, followed by the bf16 kernel as a stand-by that returns at once unless the fp16 launch
// recorded a largest |delta| outside the window in which fp16 is safe.  False: not applicable
// (fewer basis blocks, or rows for fewer than 256 workgroups: such a matrix has always had the bf16
// form), the caller goes on as usual.
static bool project_p_f16(int64_t m, int64_t n, int r, int K, const PtrPack<const float *> &delta,
                          const float *q_in, const PtrPack<float *> &out, void *workspace,
                          hipStream_t st, int *rc_out) {
    const int cb = cb_of(r);
    if (cb < 4 || out_wgs(m) * K < kQUnits) return false;
    const PPlan pl = p_plan(m, n, r, K);  // never split with that many workgroups
    const int64_t KS = ceil_div(n, 64) * 4;
    char *ws = reinterpret_cast<char *>(workspace);
    uint4 *frags2 = reinterpret_cast<uint4 *>(ws);                                // two bf16 pieces
    uint4 *frags1 = reinterpret_cast<uint4 *>(ws + (size_t)KS * cb * 2 * 1024);   // one fp16 piece
    const F16Scratch f = f16_scratch(ws + a256((size_t)KS * cb * 3 * 1024));
    int rc = pack_f16(KContig{q_in, r, n, cb, KS, frags2}, frags1, f, st);
    if (rc == DLCX_OK) {
        Timed timed(KID_PROJECT_P, st);
        if (cb == 4) {
            rc = project_p_ws_launch<1, 2, 2, 2>(pl, delta, frags1, out, m, n, r, K, st, f.record, f.out_scale);
            if (rc == DLCX_OK)
                rc = project_p_ws_launch<2, 2, 2, 2>(pl, delta, frags2, out, m, n, r, K, st, nullptr, nullptr, f.record);
        } else {
            rc = n >= kPDeep ? project_p_ws_launch<1, 2, 4, 1, 4, false, 3>(pl, delta, frags1, out, m, n, r, K, st, f.record, f.out_scale)
                             : project_p_ws_launch<1, 2, 4, 1>(pl, delta, frags1, out, m, n, r, K, st, f.record, f.out_scale);
            if (rc == DLCX_OK)
                rc = project_p_ws_launch<2, 2, 4, 1>(pl, delta, frags2, out, m, n, r, K, st, nullptr, nullptr, f.record);
        }
        if (rc == DLCX_OK) rc = check_launch("project_p_f16");
    }
    *rc_out = rc;
    return true;
}

// The sums over the splits of a reduction, left to the caller (partial) or formed here.
static int finish_splits(int K, const PartialSums &sums, const PtrPack<float *> &out,
                         PartialSums *partial, hipStream_t st) {
    if (partial) {
        *partial = sums;
        return DLCX_OK;
    }
    return launch_sum_slabs(K, sums, out, sums.stride, st);
}

template <int NS>
static int project_p_ns(int64_t m, int64_t n, int r, int K, const PtrPack<const float *> &delta,
                        const float *q_in, const PtrPack<float *> &out, void *workspace,
                        PartialSums *partial, hipStream_t st) {
    const int cb = cb_of(r);
    const PPlan pl = p_plan(m, n, r, K);
    const int64_t KS = ceil_div(n, 64) * 4, slab = (int64_t)r * m;
    char *wsb = reinterpret_cast<char *>(workspace);
    uint4 *frags = reinterpret_cast<uint4 *>(wsb);
    int rc = pack_kcontig<NS>(KContig{q_in, r, n, cb, KS, frags}, st);
    if (rc != DLCX_OK) return rc;
    PtrPack<float *> dst = out;
    PartialSums sums;
    sums.S = pl.S;
    sums.stride = slab;
    if (pl.S > 1) {
        float *base = reinterpret_cast<float *>(wsb + a256((size_t)KS * cb * NS * 1024));
        for (int k = 0; k < K; ++k) sums.slabs.p[k] = dst.p[k] = base + (int64_t)k * pl.S * slab;
    }
    {
        Timed timed(KID_PROJECT_P, st);
        switch (cb) {
            case 1:
                if (pl.one_role)
                    hipLaunchKernelGGL(project_p_one_kernel<NS>, dim3((unsigned)ceil_div(m, kOneRows), (unsigned)K),
                                       dim3(kW), 0, st, delta, frags, out, m, n, r);
                else
                    rc = project_p_ws_launch<NS, 1, 1, 4>(pl, delta, frags, dst, m, n, r, K, st);
                break;
            case 2:
                rc = pl.lone ? project_p_ws_launch<NS, 1, 2, 2, 4, true>(pl, delta, frags, dst, m, n, r, K, st)
                             : project_p_ws_launch<NS, 1, 2, 2>(pl, delta, frags, dst, m, n, r, K, st);
                break;
            case 4:
                rc = pl.rows == 64 ? project_p_ws_launch<NS, 2, 2, 2, 2>(pl, delta, frags, dst, m, n, r, K, st)
                                   : project_p_ws_launch<NS, 2, 2, 2>(pl, delta, frags, dst, m, n, r, K, st);
                break;
            default:
                rc = pl.rows == 64 ? project_p_ws_launch<NS, 2, 4, 1, 2>(pl, delta, frags, dst, m, n, r, K, st)
                                   : project_p_ws_launch<NS, 2, 4, 1>(pl, delta, frags, dst, m, n, r, K, st);
                break;
        }
        if (rc == DLCX_OK) rc = check_launch("project_p_mfma");
    }
    if (rc != DLCX_OK || pl.S == 1) return rc;
    return finish_splits(K, sums, out, partial, st);
}

template <int NS, int CBW, int WCB, bool LONE = NS == 3>
static int project_q_ws_launch(const dim3 &grid, hipStream_t st, const PtrPack<const float *> &delta,
                               const uint4 *frags, const PtrPack<float *> &dst, int64_t m,
                               int64_t n, int r, int64_t ksteps_per_wg, int64_t slab,
                               uint32_t *record = nullptr, const float *out_scale = nullptr,
                               const uint32_t *guard = nullptr) {
    constexpr int lds = 2 * 16 * NS * 1024;
    static size_t granted = 0;
    int rc = grant_dynamic_lds(reinterpret_cast<const void *>(project_q_ws_kernel<NS, CBW, WCB, LONE>),
                               lds, &granted, "project_q attribute");
    if (rc != DLCX_OK) return rc;
    hipLaunchKernelGGL((project_q_ws_kernel<NS, CBW, WCB, LONE>), grid, dim3(kWs), lds, st, delta, frags, dst,
                       m, n, r, ksteps_per_wg, slab, record, out_scale, guard);
    return DLCX_OK;
}

// F16: the fp16 form for 4 or 8 basis blocks (see project_p_f16), with the bf16 kernel as its
// stand-by; NS is then the stand-by's piece count (2) and the workspace holds three pieces.  The
// stand-by keeps the splits of DLCX_MMA_BF16, so that its result is that mode's bit for bit; which of
// the two numbers of partial sums counts is read from the record when they are added.
template <int NS, bool F16>
static int project_q_ns(int64_t m, int64_t n, int r, int K, const PtrPack<const float *> &delta,
                        const float *p_hat, const PtrPack<float *> &out, void *workspace,
                        PartialSums *partial, hipStream_t st) {
    const int cb = cb_of(r);
    const bool f16 = F16 && cb >= 4;
    const QPlan q = q_plan(NS, false, m, n, r, K), h = f16 ? q_plan(NS, true, m, n, r, K) : q;
    const int S = q.S > h.S ? q.S : h.S;  // slabs of a worker
    const int64_t KS = q.KS > h.KS ? q.KS : h.KS, slab = (int64_t)r * n;
    const int pieces = F16 ? 3 : NS;  // as the workspace was sized
    char *wsb = reinterpret_cast<char *>(workspace);
    uint4 *frags = reinterpret_cast<uint4 *>(wsb);
    uint4 *frags1 = reinterpret_cast<uint4 *>(wsb + (size_t)KS * cb * NS * 1024);
    F16Scratch f = f16_scratch(nullptr);
    int rc = DLCX_OK;
    if (f16) {
        const size_t slab_bytes = S > 1 ? a256((size_t)K * S * slab * sizeof(float)) : 0;
        f = f16_scratch(wsb + a256((size_t)KS * cb * pieces * 1024) + slab_bytes);
        rc = pack_f16(KContig{p_hat, r, m, cb, KS, frags}, frags1, f, st);
    } else {
        rc = pack_kcontig<NS>(KContig{p_hat, r, m, cb, KS, frags}, st);
    }
    if (rc != DLCX_OK) return rc;
    PtrPack<float *> dst = out;
    PartialSums sums;
    sums.S = h.S;
    sums.stride = slab;
    if (q.S != h.S) {
        sums.guard = f.record;
        sums.S_alt = q.S;
    }
    if (S > 1) {
        float *base = reinterpret_cast<float *>(wsb + a256((size_t)KS * cb * pieces * 1024));
        for (int k = 0; k < K; ++k) sums.slabs.p[k] = dst.p[k] = base + (int64_t)k * S * slab;
    }
    const dim3 grid((unsigned)out_wgs(n), (unsigned)K, (unsigned)q.S);
    const int64_t ksteps = q.ksteps_per_wave * 4;
    {
    Timed timed(KID_PROJECT_Q, st);
    if (f16) {  // the stand-by launches below then carry the record as their guard
        const dim3 hgrid(grid.x, grid.y, (unsigned)h.S);
        if (cb == 4) rc = project_q_ws_launch<1, 1, 4>(hgrid, st, delta, frags1, dst, m, n, r, h.ksteps_per_wave * 4, slab, f.record, f.out_scale);
        else rc = project_q_ws_launch<1, 2, 4>(hgrid, st, delta, frags1, dst, m, n, r, h.ksteps_per_wave * 4, slab, f.record, f.out_scale);
        if (rc != DLCX_OK) return rc;
    }
    const uint32_t *guard = f16 ? f.record : nullptr;
    switch (cb) {
        case 1:
            if constexpr (NS == 2) rc = project_q_ws_launch<NS, 1, 1>(grid, st, delta, frags, dst, m, n, r, ksteps, slab);
            else hipLaunchKernelGGL(project_q_one_kernel, grid, dim3(kW), 0, st, delta, frags, dst, m, n, r, q.ksteps_per_wave, slab);
            break;
        case 2:
            rc = q.lone ? project_q_ws_launch<NS, 1, 2, true>(grid, st, delta, frags, dst, m, n, r, ksteps, slab)
                        : project_q_ws_launch<NS, 1, 2>(grid, st, delta, frags, dst, m, n, r, ksteps, slab);
            break;
        case 4:
            rc = q.lone ? project_q_ws_launch<NS, 1, 4, true>(grid, st, delta, frags, dst, m, n, r, ksteps, slab, nullptr, nullptr, guard)
                        : project_q_ws_launch<NS, 1, 4>(grid, st, delta, frags, dst, m, n, r, ksteps, slab, nullptr, nullptr, guard);
            break;
        default: rc = project_q_ws_launch<NS, 2, 4>(grid, st, delta, frags, dst, m, n, r, ksteps, slab, nullptr, nullptr, guard); break;
    }
    if (rc == DLCX_OK) rc = check_launch("project_q_mfma");
    }
    if (rc != DLCX_OK || S == 1) return rc;
    return finish_splits(K, sums, out, partial, st);
}

int launch_project_p_mfma(int mma, int64_t m, int64_t n, int r, int K,
                          const PtrPack<const float *> &delta, const float *q_in,
                          const PtrPack<float *> &out, void *workspace, PartialSums *partial,
                          hipStream_t st) {
    if (mma == DLCX_MMA_F32)
        return project_p_ns<3>(m, n, r, K, delta, q_in, out, workspace, partial, st);
    int rc = DLCX_OK;
    if (mma == DLCX_MMA_F16 && project_p_f16(m, n, r, K, delta, q_in, out, workspace, st, &rc))
        return rc;
    return project_p_ns<2>(m, n, r, K, delta, q_in, out, workspace, partial, st);
}

int launch_project_q_mfma(int mma, int64_t m, int64_t n, int r, int K,
                          const PtrPack<const float *> &delta, const float *p_hat,
                          const PtrPack<float *> &out, void *workspace, PartialSums *partial,
                          hipStream_t st) {
    if (mma == DLCX_MMA_F32)
        return project_q_ns<3, false>(m, n, r, K, delta, p_hat, out, workspace, partial, st);
    if (mma == DLCX_MMA_F16)
        return project_q_ns<2, true>(m, n, r, K, delta, p_hat, out, workspace, partial, st);
    return project_q_ns<2, false>(m, n, r, K, delta, p_hat, out, workspace, partial, st);
}

size_t mfma_reconstruct_workspace_bytes(int mma, int64_t m, int64_t n, int r) {
    const int ns = ns_of(mma);
    const size_t ks = (size_t)(r + 15) / 16;
    return a256((size_t)ceil_div(m, 32) * ks * ns * 1024) + a256((size_t)ceil_div(n, 32) * ks * ns * 1024);
}

template <int NS>
static int reconstruct_launch(int64_t m, int64_t n, int ks, const uint4 *pf, const uint4 *qf,
                              const ReconEpilogue &ep, hipStream_t st) {
    // Columns per workgroup: one 32 x 256 tile each, workgroups in tile order along the row block.
    // This kernel leaves no partial sums behind, so nothing speaks for longer column ranges, and
    // short ranges in tile order are what the memory system likes best (measured at rank 200:
    // 28672 x 8192 5.08 -> 5.63 TB/s against ranges of 1792 columns, 8192 x 28672 4.85 -> 5.12,
    // 8192 x 8192 5.2 -> 5.45; one or two long ranges per row block: 3.0 - 4.6).
    const int64_t rows = ceil_div(m, 32);
    const int64_t cols = 256;
    const dim3 grid((unsigned)ceil_div(n, cols), (unsigned)rows);
    Timed timed(KID_RECONSTRUCT, st);
    hipLaunchKernelGGL(reconstruct_mfma_kernel<NS>, grid, dim3(kW), 0, st, pf, qf, ep, m, n, cols,
                       ks);
    return check_launch("reconstruct_mfma");
}

template <int NS>
static int reconstruct_ns(int64_t m, int64_t n, int r, const float *p_hat, const float *q_bar,
                          const ReconEpilogue &ep, void *workspace, hipStream_t st) {
    const int ks = (r + 15) / 16;
    const int64_t xbm = ceil_div(m, 32), xbn = ceil_div(n, 32);
    uint4 *pf = reinterpret_cast<uint4 *>(workspace);
    uint4 *qf = reinterpret_cast<uint4 *>(reinterpret_cast<char *>(workspace) +
                                          a256((size_t)xbm * ks * NS * 1024));
    const int rc = pack_sweep<NS>(KContig{}, KStrided{p_hat, r, m, ks, xbm, pf},
                                  KStrided{q_bar, r, n, ks, xbn, qf}, st);
    if (rc != DLCX_OK) return rc;
    return reconstruct_launch<NS>(m, n, ks, pf, qf, ep, st);
}

int launch_reconstruct_mfma(int mma, int64_t m, int64_t n, int r, const float *p_hat,
                            const float *q_bar, const ReconEpilogue &ep, void *workspace,
                            hipStream_t st) {
    if (mma == DLCX_MMA_F32) return reconstruct_ns<3>(m, n, r, p_hat, q_bar, ep, workspace, st);
    return reconstruct_ns<2>(m, n, r, p_hat, q_bar, ep, workspace, st);
}

// ---- fused round: workspace layout and launch ------------------------------------------------
constexpr int kComputeUnits = 256;
struct RoundPlan {
    int chunks;  // column ranges per row block = slabs per worker
    int tiles;   // 256-column tiles of a row block; range x starts at tile ceil(x tiles / chunks)
    int kc;      // workers per launch
};

// Column ranges per row block.  One workgroup fills a compute unit, so the launch takes as many
// rounds as it has workgroups for each of the 256 units, and a round as long as its longest range
// plus about 0.3 tiles of start-up and of slab: the cheapest count by that estimate.  Against the
// counts measured (1 .. all tiles, us, chosen | rule before: 4 ranges from 2048 columns on, ranges of
// 512 columns or more, at most 8): 5008 x 3376 three workers 3 ranges 274 | 4: 312; 8192 x 2048 1:
// 205 | 4: 241; 8192 x 1024 1: 111 | 2: 125; 704 x 4160 9: 50 | 6: 61; 512 x 8192 16: 63 | 8: 79; 3008
// x 6000 8: 309 | 6: 357; 512 x 512 2: 20 | 1: 23; 2048 x 8192 4: 194.  No ranges of more than 8 tiles
// up to four ranges: one or two long ones are 13 % slower at 8192 columns whatever the number of rows
// (the workgroups drift apart), and the count does not matter at 28672.  At 4096 columns two ranges are
// already too long: 4096 x 4096 r = 32 two workers 191, three 158, four 137; 11008 x 4096 467 | 366 | 355,
// eight 338; 8192 x 4096 324 | 265 | 253.  (3840 and 4080 columns: two are as good as four.)
static RoundPlan round_plan(int64_t m, int64_t n) {
    RoundPlan p;
    p.kc = 4;  // workers per launch: 4 x 2 basis blocks x 16 accumulator registers per wavefront
    const int64_t rows = ceil_div(m, 32), tiles = ceil_div(n, 256);
    const int64_t lo = tiles > 24 ? 4 : n == 4096 ? 3 : ceil_div(tiles, 8), hi = tiles < 32 ? tiles : 32;
    int64_t best = lo, best_cost = INT64_MAX;
    for (int64_t c = lo; c <= hi; ++c) {
        const int64_t cost = ceil_div(rows * c, kComputeUnits) * (10 * ceil_div(tiles, c) + 3);
        if (cost < best_cost) {
            best = c;
            best_cost = cost;
        }
    }
    p.chunks = (int)best;
    p.tiles = (int)tiles;
    return p;
}

// [basis fragments | P_hat_prev fragments | Q_bar_prev fragments | slabs (K x chunks x r x m)]
size_t mfma_round_workspace_bytes(int mma, int64_t m, int64_t n, int r, int r_prev, int K) {
    const int ns = ns_of(mma);
    const RoundPlan pl = round_plan(m, n);
    const size_t ksp = (size_t)(r_prev + 15) / 16;
    size_t total = a256((size_t)ceil_div(n, 64) * 4 * cb_of(r) * ns * 1024);
    total += a256((size_t)ceil_div(m, 32) * ksp * ns * 1024);
    total += a256((size_t)ceil_div(n, 32) * ksp * ns * 1024);
    if (pl.chunks > 1) total += a256((size_t)K * pl.chunks * r * m * sizeof(float));
    return total;
}

template <int NS, int CB, int KC, bool TLBF16>
static int round_launch_t(const uint4 *pf, const uint4 *qf, int ks, const uint4 *bf,
                        const ReconEpilogue &ep, const PtrPack<float *> &pslab, int64_t m,
                        int64_t n, int r, const RoundPlan &pl, int64_t slab_stride,
                        hipStream_t st) {
    const size_t tiles = 4 * (size_t)round_tile_bytes(NS) + 4 * (size_t)(4 * CB * NS * 1024);
    const size_t red = (size_t)KC * CB * 16 * 64 * 4;
    const size_t lds = tiles > red ? tiles : red;
    static size_t granted = 0;
    int rc = grant_dynamic_lds(reinterpret_cast<const void *>(round_mfma_kernel<NS, CB, KC, TLBF16>),
                               lds, &granted, "round kernel attribute");
    if (rc != DLCX_OK) return rc;
    const dim3 grid((unsigned)pl.chunks, (unsigned)ceil_div(m, 32));
    Timed timed(KID_ROUND, st);
    hipLaunchKernelGGL((round_mfma_kernel<NS, CB, KC, TLBF16>), grid, dim3(kW), lds, st, pf, qf, ks,
                       bf, ep, pslab, m, n, r, pl.tiles, slab_stride);
    return check_launch("round_mfma");
}

template <int NS, int CB, int KC>
static int round_launch(const uint4 *pf, const uint4 *qf, int ks, const uint4 *bf,
                        const ReconEpilogue &ep, const PtrPack<float *> &pslab, int64_t m,
                        int64_t n, int r, const RoundPlan &pl, int64_t slab_stride,
                        hipStream_t st) {
    if (ep.tl_bf16)
        return round_launch_t<NS, CB, KC, true>(pf, qf, ks, bf, ep, pslab, m, n, r, pl, slab_stride, st);
    return round_launch_t<NS, CB, KC, false>(pf, qf, ks, bf, ep, pslab, m, n, r, pl, slab_stride, st);
}

template <int NS>
static int round_ns(int64_t m, int64_t n, int r, int r_prev, const float *p_hat, const float *q_bar,
                    const float *basis, const ReconEpilogue &ep_all, const PtrPack<float *> &factors,
                    void *workspace, PartialSums *partial, hipStream_t st) {
    const int cb = cb_of(r);
    const RoundPlan pl = round_plan(m, n);
    const int ks = (r_prev + 15) / 16;
    const int64_t xbm = ceil_div(m, 32), xbn = ceil_div(n, 32);
    char *ws = reinterpret_cast<char *>(workspace);
    uint4 *bf = reinterpret_cast<uint4 *>(ws);
    ws += a256((size_t)ceil_div(n, 64) * 4 * cb * NS * 1024);
    uint4 *pf = reinterpret_cast<uint4 *>(ws);
    ws += a256((size_t)xbm * ks * NS * 1024);
    uint4 *qf = reinterpret_cast<uint4 *>(ws);
    ws += a256((size_t)xbn * ks * NS * 1024);
    float *slabs = reinterpret_cast<float *>(ws);
    // (r_prev == 0: no factors to pack)
    int rc = pack_sweep<NS>(KContig{basis, r, n, cb, ceil_div(n, 64) * 4, bf},
                            KStrided{p_hat, r_prev, m, ks, ks > 0 ? xbm : 0, pf},
                            KStrided{q_bar, r_prev, n, ks, ks > 0 ? xbn : 0, qf}, st);
    if (rc != DLCX_OK) return rc;
    const int64_t slab = (int64_t)r * m;
    for (int k0 = 0; k0 < ep_all.K; k0 += pl.kc) {
        ReconEpilogue ep = ep_all;
        ep.K = ep_all.K - k0 < pl.kc ? ep_all.K - k0 : pl.kc;
        ep.apply = ep_all.apply && (k0 + pl.kc >= ep_all.K);  // theta moves with the last group
        PtrPack<float *> dst;
        for (int k = 0; k < ep.K; ++k) {
            ep.ef.p[k] = ep_all.ef.p[k0 + k];
            ep.tl.p[k] = ep_all.tl.p[k0 + k];
            dst.p[k] = pl.chunks > 1 ? slabs + (int64_t)(k0 + k) * pl.chunks * slab
                                     : factors.p[k0 + k];
        }
        switch (cb) {  // ranks above 64 do not come here: see dlcx_ef_delta_apply_compress
            case 1: rc = round_launch<NS, 1, 4>(pf, qf, ks, bf, ep, dst, m, n, r, pl, slab, st); break;
            case 2: rc = round_launch<NS, 2, 4>(pf, qf, ks, bf, ep, dst, m, n, r, pl, slab, st); break;
            default: rc = DLCX_EINVAL; break;
        }
        if (rc != DLCX_OK) return rc;
    }
    partial->S = pl.chunks;
    partial->stride = slab;
    for (int k = 0; k < ep_all.K; ++k) partial->slabs.p[k] = slabs + (int64_t)k * pl.chunks * slab;
    return DLCX_OK;
}

int launch_round_mfma(int mma, int64_t m, int64_t n, int r, int r_prev, const float *p_hat,
                      const float *q_bar, const float *basis, const ReconEpilogue &ep,
                      const PtrPack<float *> &factors, void *workspace, PartialSums *partial,
                      hipStream_t st) {
    if (mma == DLCX_MMA_F32)
        return round_ns<3>(m, n, r, r_prev, p_hat, q_bar, basis, ep, factors, workspace, partial,
                           st);
    return round_ns<2>(m, n, r, r_prev, p_hat, q_bar, basis, ep, factors, workspace, partial,
                           st);
}

}  // namespace dlcx
