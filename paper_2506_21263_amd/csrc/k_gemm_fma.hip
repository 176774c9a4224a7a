// Rank-r products of the low-rank compressor with fp32 operands and fp64 accumulation
// (DLCX_MMA_FMA): the accuracy mode, the GPU path whose rounding is closest to the exact products
// (a product of two fp32 values is exact in fp64), for every shape the interface allows.  They run
// on v_mfma_f64_16x16x4_f64, at 1/32 of the bf16 rate, which bounds them from
// about rank 16 on; the modes with split operands live in k_gemm_mfma.hip.
//
// Operands of that instruction, lane l with g = l / 16, n = l % 16: A[n][g], B[g][n], result
// D[4 v + g][n] in register v.  Where the reduction index is contiguous in memory a lane loads four
// consecutive values and feeds one to each of four products (both operands agree on that order of
// the reduction), where the other index is contiguous it loads four columns and feeds one to each
// of four column blocks, 4 n + q being column n of block q: all loads are 16 bytes a lane, go
// straight to registers and are requested a step ahead.  Every side is a multiple of 16.
#include <type_traits>

#include "common.h"

namespace dlcx {

constexpr int kT = 256;  // threads per workgroup (4 wavefronts)

__device__ __forceinline__ f64x4_t mfma64(float a, float b, f64x4_t c) { return mfma64((double)a, (double)b, c); }
__device__ __forceinline__ float part_of(const float4 &v, int s) {
    return s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w;
}
__device__ __forceinline__ float4 load4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
// What was requested before this stays before the products behind it.
template <bool kOrdered>
__device__ __forceinline__ void keep_order() {
    if constexpr (kOrdered) __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------------------------
// P_k = delta_k * Q_in:  D[c][i] = sum_j Q[c][j] delta[i][j].  Workgroup: 16 RB rows of delta and
// all r outputs; each wavefront sums a quarter of the columns j, the four sums are added in order.
// (One wavefront per row group and no split leaves most SIMDs idle below 16 K rows.)
// 2048 x 2048, four workers, r = 32: 27 us with the quantiser (scalar fp64 FMAs on LDS operands: 693 us); the
// matrix cores' own time is 14 us.  kAhead sets of operands are requested before the one that is multiplied.  Two
// for long reductions, and the requests do not sink behind products: with one set ahead, left to the compiler, 33
// us; 2480 x 2480 five workers r = 64 120 | 107, 2048 x 2048 four r = 100 94 | 77, two r = 200 108 | 89 (one set
// ahead there, in order: registers).  One, left to the compiler, for short ones (p_sets_ahead).
// ---------------------------------------------------------------------------------------------
template <int CB, int RB, int kAhead>
__global__ __launch_bounds__(kT) void project_p_f64_kernel(PtrPack<const float *> deltas,
                                                           const float *__restrict__ q_in,
                                                           PtrPack<float *> outs, int64_t m,
                                                           int64_t n, int r) {
    constexpr int U = CB <= 4 ? 2 : 1;  // steps of 16 columns per set of operands
    constexpr bool kOrdered = kAhead > 1 || CB > 8;
    __shared__ double red[4][RB * 4][64];
    const float *__restrict__ delta = deltas.p[blockIdx.y];
    float *__restrict__ out = outs.p[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, x = lane & 15;
    const int64_t i0 = (int64_t)blockIdx.x * (16 * RB);
    const int64_t steps = n >> 4, per = (steps + 3) >> 2;
    const int64_t begin = wave * per, end = begin + per < steps ? begin + per : steps;

    const float *pd[RB], *pq[CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {  // past the last row, or the last column of the factor: any
        const int64_t i = i0 + rb * 16 < m ? i0 + rb * 16 + x : x;  // valid one, nothing is stored
        pd[rb] = delta + i * n + 4 * g;
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int c = cb * 16 + x;
        pq[cb] = q_in + (int64_t)(c < r ? c : r - 1) * n + 4 * g;
    }
    f64x4_t acc[CB][RB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[cb][rb] = f64x4_t{0.0, 0.0, 0.0, 0.0};

    struct Set {
        float4 a[U][CB], b[U][RB];
    };
    auto load = [&](Set &s, int64_t step) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t st = step + u < end ? step + u : end - 1;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) s.b[u][rb] = load4(pd[rb] + st * 16);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                if (cb * 16 < r) s.a[u][cb] = load4(pq[cb] + st * 16);
        }
    };
    auto multiply = [&](const Set &cur, int64_t st) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (st + u >= end) break;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                if (cb * 16 < r) {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb)
                            acc[cb][rb] = mfma64(part_of(cur.a[u][cb], s), part_of(cur.b[u][rb], s), acc[cb][rb]);
                }
        }
        keep_order<kOrdered>();
    };
    if (begin < end) {
        Set set[kAhead + 1];
#pragma unroll
        for (int d = 0; d < kAhead; ++d) load(set[d], begin + d * U);
        for (int64_t st = begin; st < end; st += (kAhead + 1) * U)
#pragma unroll
            for (int d = 0; d <= kAhead; ++d) {
                if (st + d * U >= end) break;
                load(set[(d + kAhead) % (kAhead + 1)], st + (d + kAhead) * U);
                keep_order<kOrdered>();
                multiply(set[d], st + d * U);
            }
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        if (cb * 16 >= r) break;
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][rb * 4 + v][lane] = acc[cb][rb][v];
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {  // wavefront v adds register v of the four
            const int e = rb * 4 + wave, c = cb * 16 + 4 * wave + g;
            const int64_t i = i0 + rb * 16 + x;
            const double s = ((red[0][e][lane] + red[1][e][lane]) + red[2][e][lane]) + red[3][e][lane];
            if (c < r && i < m) out[(int64_t)c * m + i] = (float)s;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Q_k = delta_k^T * P_hat:  D[c][j] = sum_i P_hat[c][i] delta[i][j].  Workgroup: 64 columns of delta
// over the row range of split blockIdx.z; partial results go to slab blockIdx.z (summed afterwards
// in slab order).  The wavefronts are WC groups of CBW blocks of outputs by WK = 4 / WC quarters or
// halves of the rows, added in order.  2048 x 2048, four workers, r = 32: 30 us with
// the quantiser (scalar fp64 FMAs on LDS operands: 114 us).  Operands as in the P kernel.
// ---------------------------------------------------------------------------------------------
template <int CBW, int WC, int kAhead>
__global__ __launch_bounds__(kT) void project_q_f64_kernel(PtrPack<const float *> deltas,
                                                           const float *__restrict__ p_hat,
                                                           PtrPack<float *> outs, int64_t m,
                                                           int64_t n, int r, int64_t rows_per_split,
                                                           int64_t slab_stride) {
    constexpr int WK = 4 / WC;
    __shared__ double red[4][16][64];
    const float *__restrict__ delta = deltas.p[blockIdx.y];
    float *__restrict__ out = outs.p[blockIdx.y] + (int64_t)blockIdx.z * slab_stride;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, x = lane & 15;
    const int wc = wave % WC, wk = wave / WC;
    const int64_t j = (int64_t)blockIdx.x * 64 + 4 * x;
    const int cfirst = wc * CBW * 16;
    // this wavefront's rows: multiples of 16 inside the split (rows_per_split is one of 64)
    const int64_t share = rows_per_split / WK;
    const int64_t begin = (int64_t)blockIdx.z * rows_per_split + wk * share;
    const int64_t end = begin + share < m ? begin + share : m;

    const float *pd = delta + (4 * g) * n + (j < n ? j : 0);
    const float *pp[CBW];
#pragma unroll
    for (int cb = 0; cb < CBW; ++cb) {
        const int c = cfirst + cb * 16 + x;
        pp[cb] = p_hat + (int64_t)(c < r ? c : r - 1) * m + 4 * g;
    }
    f64x4_t acc[CBW][4];
#pragma unroll
    for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[cb][q] = f64x4_t{0.0, 0.0, 0.0, 0.0};

    struct Set {
        float4 a[CBW], b[4];
    };
    auto load = [&](Set &s, int64_t i) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s.b[u] = load4(pd + (i + u) * n);
#pragma unroll
        for (int cb = 0; cb < CBW; ++cb)
            if (cfirst + cb * 16 < r) s.a[cb] = load4(pp[cb] + i);
    };
    if (begin < end) {
        Set set[kAhead + 1];
#pragma unroll
        for (int d = 0; d < kAhead; ++d) load(set[d], begin + 16 * d < end ? begin + 16 * d : begin);
        for (int64_t first = begin; first < end; first += 16 * (kAhead + 1))
#pragma unroll
            for (int d = 0; d <= kAhead; ++d) {
                const int64_t i = first + 16 * d, then = i + 16 * kAhead;
                if (i >= end) break;
                load(set[(d + kAhead) % (kAhead + 1)], then < end ? then : i);
                keep_order<(kAhead > 1)>();
#pragma unroll
                for (int cb = 0; cb < CBW; ++cb)
                    if (cfirst + cb * 16 < r) {
#pragma unroll
                        for (int s = 0; s < 4; ++s)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                acc[cb][q] = mfma64(part_of(set[d].a[cb], s), part_of(set[d].b[s], q), acc[cb][q]);
                    }
                keep_order<(kAhead > 1)>();
            }
    }
#pragma unroll
    for (int cb = 0; cb < CBW; ++cb) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][v * 4 + q][lane] = acc[cb][q][v];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4 / WK; ++u) {  // registers v of this wavefront's share, all four blocks q
            const int v = wk * (4 / WK) + u, c = cfirst + cb * 16 + 4 * v + g;
            float o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                double s = red[wc][v * 4 + q][lane];
#pragma unroll
                for (int k = 1; k < WK; ++k) s += red[k * WC + wc][v * 4 + q][lane];
                o[q] = (float)s;
            }
            if (c < r && j < n)
                *reinterpret_cast<float4 *>(out + (int64_t)c * n + j) = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
}

// out[k][x] = sum_s slabs[k][s][x], s in index order (fixed order: run-to-run identical)
__global__ __launch_bounds__(kT) void sum_slabs_kernel(PtrPack<const float *> slabs,
                                                       PtrPack<float *> outs, int64_t nvec,
                                                       int64_t slab_stride, int S, int S_alt,
                                                       const uint32_t *guard) {
    const int64_t v = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (v >= nvec) return;
    reinterpret_cast<float4 *>(outs.p[blockIdx.y])[v] =
        sum_partials(slabs.p[blockIdx.y], slab_stride, split_count(S, S_alt, guard), v);
}

int launch_sum_slabs(int K, const PartialSums &part, const PtrPack<float *> &outs, int64_t count,
                     hipStream_t st) {
    const int64_t nvec = count >> 2;
    Timed timed(KID_SUM_SLABS, st);
    hipLaunchKernelGGL(sum_slabs_kernel, dim3((unsigned)ceil_div(nvec, kT), (unsigned)K), dim3(kT),
                       0, st, part.slabs, outs, nvec, part.stride, part.S, part.S_alt, part.guard);
    return check_launch("sum_slabs");
}

// ---------------------------------------------------------------------------------------------
// delta_hat = P_hat Q_bar^T:  D[i][j] = sum_c P_hat[c][i] Q_bar[c][j], 16 rows x 64 columns per
// wavefront (WC wavefronts of a workgroup beside one another, 4 / WC below), so that a lane ends up
// with four consecutive columns of four rows; the epilogue writes the tile (optional), subtracts it from the K error buffers (e_k <-
// delta_k - delta_hat) and, when theta is given, forms the next pseudo-gradients and applies the
// Nesterov outer update with the tile as the gradient.
// ---------------------------------------------------------------------------------------------
template <int WC>
__global__ __launch_bounds__(kT) void reconstruct_f64_kernel(const float *__restrict__ p_hat,
                                                             const float *__restrict__ q_bar,
                                                             ReconEpilogue ep, int64_t m,
                                                             int64_t n, int r, int col_wgs) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, x = lane & 15;
    const int64_t i0 = (int64_t)(blockIdx.x / col_wgs) * (64 / WC) + wave / WC * 16;
    const int64_t j = (int64_t)(blockIdx.x % col_wgs) * (64 * WC) + wave % WC * 64 + 4 * x;
    if (i0 >= m) return;
    const float *pa = p_hat + i0 + x, *pb = q_bar + (j < n ? j : 0);
    f64x4_t acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    struct Set {
        float a[4];
        float4 b[4];
    };
    auto load = [&](Set &s, int c0) {  // columns c0 .. c0 + 15 of the factors, zeros from r on
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + 4 * u + g, cc = c < r ? c : r - 1;
            const float a = pa[(int64_t)cc * m];
            s.b[u] = load4(pb + (int64_t)cc * n);
            s.a[u] = c < r ? a : 0.f;
            if (c >= r) s.b[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    Set cur, next;
    load(cur, 0);
    for (int c0 = 0; c0 < r; c0 += 16) {
        load(next, c0 + 16);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = mfma64(cur.a[u], part_of(cur.b[u], q), acc[q]);
        cur = next;
    }
    if (j >= n) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int64_t off = (i0 + 4 * v + g) * n + j;
        const float4 d = make_float4((float)acc[0][v], (float)acc[1][v], (float)acc[2][v],
                                     (float)acc[3][v]);
        if (ep.out) *reinterpret_cast<float4 *>(ep.out + off) = d;
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f), vel = t;
        if (ep.tl_on || ep.apply) t = load4(ep.theta + off);
        if (ep.apply) vel = load4(ep.vel + off);
        for (int k0 = 0; k0 < ep.K; k0 += 4) {  // four workers' loads before the first store
            float4 e[4], l[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (k0 + k >= ep.K) break;
                e[k] = load4(ep.ef.p[k0 + k] + off);
                if (ep.tl_on && ep.tl_bf16) {
                    const uint2 b = *reinterpret_cast<const uint2 *>(
                        reinterpret_cast<const uint16_t *>(ep.tl.p[k0 + k]) + off);
                    l[k] = make_float4(__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xFFFF0000u),
                                       __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xFFFF0000u));
                } else if (ep.tl_on) {
                    l[k] = load4(reinterpret_cast<const float *>(ep.tl.p[k0 + k]) + off);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (k0 + k >= ep.K) break;
                float4 y = e[k];
                y.x -= d.x; y.y -= d.y; y.z -= d.z; y.w -= d.w;
                if (ep.tl_on) {
                    y.x = (t.x - l[k].x) + y.x; y.y = (t.y - l[k].y) + y.y;
                    y.z = (t.z - l[k].z) + y.z; y.w = (t.w - l[k].w) + y.w;
                }
                *reinterpret_cast<float4 *>(ep.ef.p[k0 + k] + off) = y;
            }
        }
        if (ep.apply) {
            vel.x = fmaf(ep.mu, vel.x, d.x); vel.y = fmaf(ep.mu, vel.y, d.y);
            vel.z = fmaf(ep.mu, vel.z, d.z); vel.w = fmaf(ep.mu, vel.w, d.w);
            t.x = fmaf(-ep.lr, fmaf(ep.mu, vel.x, d.x), t.x);
            t.y = fmaf(-ep.lr, fmaf(ep.mu, vel.y, d.y), t.y);
            t.z = fmaf(-ep.lr, fmaf(ep.mu, vel.z, d.z), t.z);
            t.w = fmaf(-ep.lr, fmaf(ep.mu, vel.w, d.w), t.w);
            *reinterpret_cast<float4 *>(ep.vel + off) = vel;
            *reinterpret_cast<float4 *>(ep.theta + off) = t;
        }
    }
}

// ---------------------------------------------------------------------------------------------
static int q_splits(int64_t m, int64_t n, int K) {
    const int64_t wgs = ceil_div(n, 64) * K;
    int64_t s = ceil_div(1024, wgs);
    const int64_t smax = ceil_div(m, 256);
    if (s > smax) s = smax;
    if (s > 64) s = 64;
    return (int)(s < 1 ? 1 : s);
}

size_t fma_project_workspace_bytes(int64_t m, int64_t n, int r, int K) {
    // Q phase: slabs of r x n floats, enough for any smaller number of workers that is later run in this
    // workspace: fewer workers may be split further, 8 at 8256 columns not at all, 7 in two (14 slabs)
    int64_t slabs = 0;
    for (int k = 1; k <= K; ++k) {
        const int64_t s = (int64_t)k * q_splits(m, n, k);
        if (s > slabs) slabs = s;
    }
    return (size_t)slabs * (size_t)r * (size_t)n * sizeof(float);
}

// Sets of operands that a wavefront of the P kernel requests ahead, at ranks up to 64.  A wavefront has a quarter of
// the n / 16 steps: up to 768 columns two sets are most of it and the registers they take cost more than they hide;
// with one basis block and more than one workgroup of two row blocks to a unit, up to 2048 columns, other wavefronts
// hide what one set leaves.  One | two, us: 2480 x 192 eight workers r = 9 7.9 | 9.6, 688 x 256 three r = 16 4.3 | 4.5,
// 4800 x 768 eight r = 32 41.9 | 44.1, 2480 x 2048 eight r = 16 39.1 | 40.7; 1264 x 1024 five r = 17 15.7 | 14.4, 1264
// x 2048 five r = 32 27.6 | 24.8, 2480 x 4096 eight r = 48 186 | 175.
static int p_sets_ahead(int64_t n, int r, int64_t pairs) { return n <= 768 || (r <= 16 && pairs > 256 && n <= 2048) ? 1 : 2; }

int launch_project_p_fma(int64_t m, int64_t n, int r, int K, const PtrPack<const float *> &delta,
                         const float *q_in, const PtrPack<float *> &out, hipStream_t st) {
    Timed timed(KID_PROJECT_P, st);
    auto go = [&](auto cb, auto rb, auto ahead) {
        const dim3 grid((unsigned)ceil_div(m, 16 * decltype(rb)::value), (unsigned)K);
        hipLaunchKernelGGL((project_p_f64_kernel<decltype(cb)::value, decltype(rb)::value, decltype(ahead)::value>),
                           grid, dim3(kT), 0, st, delta, q_in, out, m, n, r);
    };
    typedef std::integral_constant<int, 1> one;
    typedef std::integral_constant<int, 2> two;
    // Two row blocks to a workgroup, half as many conversions and basis operands to a product, take nine tenths of the
    // time of two workgroups with one, if as many units are busy: rounds of the launch on 256 units, by either kind,
    // while one round or two is all there is: one round of pairs for two of singles (129 .. 256 pairs), two for four
    // (from 385 on).  One | two, us, four workers (five at 2480): 128 pairs 1024 x 2000 r = 8 11.6 | 15.0, r = 48 25.4 |
    // 34.8; 136 .. 256 pairs 1088 x 512 r = 8 6.5 | 6.1, r = 64 15.8 | 15.7, 1088 x 2000 r = 1 14.7 | 15.1, r = 16 15.8 |
    // 15.4, r = 64 44.9 | 45.1, 1616 x 8192 r = 16 61.0 | 50.0, 2048 x 8192 r = 32 105 | 83; 260 pairs 2064 x 2000 r = 16
    // 21.3 | 23.1, r = 64 69.9 | 74.8; 390 .. 512 pairs 2480 x 2000 r = 16 27.5 | 23.6, r = 64 84.1 | 76.5, 4080 x 2000 r =
    // 32 46.5 | 42.2.
    const int64_t pairs = ceil_div(m, 32) * K, singles = ceil_div(m, 16) * K;
    const bool pair = pairs >= 512 || 2 * ceil_div(pairs, 256) * 9 <= ceil_div(singles, 256) * 10;
    const bool far = p_sets_ahead(n, r, pairs) > 1;
    auto rows = [&](auto cb) {
        if (pair) far ? go(cb, two(), two()) : go(cb, two(), one());
        else far ? go(cb, one(), two()) : go(cb, one(), one());
    };
    if (r <= 16) rows(one());
    else if (r <= 32) rows(two());
    else if (r <= 64) rows(std::integral_constant<int, 4>());
    else if (r <= 128) go(std::integral_constant<int, 8>(), one(), two());
    else go(std::integral_constant<int, 16>(), one(), one());
    return check_launch("project_p_f64");
}

int launch_project_q_fma(int64_t m, int64_t n, int r, int K, const PtrPack<const float *> &delta,
                         const float *p_hat, const PtrPack<float *> &out, void *workspace,
                         PartialSums *partial, hipStream_t st) {
    const int64_t rows = ceil_div(ceil_div(m, q_splits(m, n, K)), 64) * 64;
    const int S = (int)ceil_div(m, rows);  // no more than q_splits: the slabs fit
    const int64_t slab = (int64_t)r * n;
    PtrPack<float *> dst = out;
    if (S > 1)
        for (int k = 0; k < K; ++k) dst.p[k] = reinterpret_cast<float *>(workspace) + (int64_t)k * S * slab;
    int rc;
    {
        Timed timed(KID_PROJECT_Q, st);
        auto launch = [&](auto cbw, auto wc, auto ahead) {
            const dim3 grid((unsigned)ceil_div(n, 64), (unsigned)K, (unsigned)S);
            hipLaunchKernelGGL((project_q_f64_kernel<decltype(cbw)::value, decltype(wc)::value, decltype(ahead)::value>),
                               grid, dim3(kT), 0, st, delta, p_hat, dst, m, n, r, rows, slab);
        };
        typedef std::integral_constant<int, 1> one;
        typedef std::integral_constant<int, 2> two;
        typedef std::integral_constant<int, 4> four;
        // Sets of operands requested ahead: two from more than 512 rows to a workgroup on and above rank 128, never
        // with one block of outputs.  One | two, us: 64 x 1072 three workers r = 64 6.8 | 7.4, 2480 x 2480 five r = 32
        // 48.4 | 50.7, 8192 x 8192 r = 16 49.5 | 53.4; 8192 x 8192 r = 32 79.5 | 77.7, r = 64 177 | 165, 2480 x 2480 five
        // r = 200 310 | 300.
        auto go = [&](auto cbw, auto wc) { rows > 512 ? launch(cbw, wc, two()) : launch(cbw, wc, one()); };
        if (r <= 16) launch(one(), one(), one());
        else if (r <= 32) go(two(), one());
        else if (r <= 64) go(four(), one());
        else if (r <= 128) go(four(), two());
        else launch(four(), four(), two());
        rc = check_launch("project_q_f64");
    }
    if (rc != DLCX_OK || S == 1) return rc;
    PartialSums sums;
    sums.S = S;
    sums.stride = slab;
    for (int k = 0; k < K; ++k) sums.slabs.p[k] = dst.p[k];
    if (partial) {
        *partial = sums;
        return DLCX_OK;
    }
    return launch_sum_slabs(K, sums, out, slab, st);
}

int launch_reconstruct_fma(int64_t m, int64_t n, int r, const float *p_hat, const float *q_bar,
                           const ReconEpilogue &ep, hipStream_t st) {
    Timed timed(KID_RECONSTRUCT, st);
    auto go = [&](auto wc) {  // the grid in one dimension: m / 16 may exceed the others'
        constexpr int WC = decltype(wc)::value;
        const int64_t col_wgs = ceil_div(n, 64 * WC);
        const dim3 grid((unsigned)(col_wgs * ceil_div(m, 64 / WC)));
        hipLaunchKernelGGL(reconstruct_f64_kernel<WC>, grid, dim3(kT), 0, st, p_hat, q_bar, ep, m, n, r,
                           (int)col_wgs);
    };
    // no wavefront without columns: 8192 x 64 r = 64 11.1 us, four side by side 12.4
    if (n <= 64) go(std::integral_constant<int, 1>());
    else if (n <= 128) go(std::integral_constant<int, 2>());
    else go(std::integral_constant<int, 4>());
    return check_launch("reconstruct_f64");
}

}  // namespace dlcx
