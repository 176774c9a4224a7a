// Shared host/device declarations of the dlcx HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <type_traits>

#include "../../include/dlcx.h"

namespace dlcx {

// K device pointers passed to a kernel by value.
template <typename T>
struct PtrPack {
    T p[DLCX_MAX_WORKERS];
};

// Records a HIP error for dlcx_last_hip_error(); returns DLCX_ELAUNCH or DLCX_OK.
int note_hip(hipError_t e, const char *where);

inline int check_launch(const char *where) { return note_hip(hipGetLastError(), where); }

// Raises `kernel`'s limit of dynamic LDS to at least `bytes` (needed above 48 KB).  *granted
// remembers the largest value set so far for that kernel; check, call and update happen under
// one process-wide lock, so two host threads that launch on two streams can neither skip a
// needed call nor leave a smaller limit behind a larger request.
int grant_dynamic_lds(const void *kernel, size_t bytes, size_t *granted, const char *what);

// Optional per-kernel timing (dlcx_profile_*): when enabled, a Timed object brackets one kernel
// launch with two HIP events on the launch stream.  Off by default; costs nothing when off.
enum KernelId {
    KID_DELTA_EF = 0, KID_NESTEROV, KID_QUANTIZE, KID_DEQUANT_AVG, KID_PACK, KID_PROJECT_P,
    KID_PROJECT_Q, KID_SUM_SLABS, KID_RECONSTRUCT, KID_GRAM, KID_CHOL, KID_APPLY_W, KID_EFF_RANK,
    KID_ROUND, KID_QUANT_ROUND, KID_REQUANT, KID_EF_UPDATE,
    KID_MFMA_PEAK, KID_TRAFFIC_PROBE, KID_COUNT
};
struct Timed {
    Timed(int kid, hipStream_t st);
    ~Timed();
    int slot;
    hipStream_t st;
    void *stop;  // the closing event of this launch's record
};

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// ---- streaming kernels (k_stream.hip) -------------------------------------------------
int launch_delta_ef(const float *theta_g, const void *theta_l, int dtype, float *ef,
                    int64_t numel, hipStream_t st);
int launch_nesterov(float *theta, float *v, const float *g, int64_t numel, float lr, float mu,
                    hipStream_t st);

// ---- quantiser (k_quant.hip) ----------------------------------------------------------
// K factors of `count` floats each; x.p[k] -> codes.p[k], scales.p[k].
int launch_quantize(int K, const PtrPack<const float *> &x, int64_t count, int qbits, int group,
                    const PtrPack<uint8_t *> &codes, const PtrPack<float *> &scales,
                    hipStream_t st, float *mean = nullptr);
// The same on sums that are still partial: x[k] = sum_s slabs[k][s] in slab order (S slabs `stride`
// floats apart) is written to sums.p[k] and quantised in one pass.
struct PartialSums {
    int S = 1;  // 1 without a guard: nothing to add, the sums are where they belong
    int64_t stride = 0;
    PtrPack<const float *> slabs;
    // Sums of an fp16 launch and its stand-by, which may have been split differently: there are S of
    // them if the record that `guard` points to says that the fp16 launch counts, else S_alt.
    const uint32_t *guard = nullptr;
    int S_alt = 1;
};
// Did the fp16 form of a projection see its operands in range?  (largest |delta| as fp32 bits)
__device__ __forceinline__ bool f16_range_ok(uint32_t amax_bits) {
    const float a = __uint_as_float(amax_bits);
    return a >= 0x1p-14f && a < 15.99f;
}
// (A kernel takes the members one by one: the whole struct, indexed by worker, would go to scratch.)
__device__ __forceinline__ int split_count(int S, int S_alt, const uint32_t *guard) {
    return guard != nullptr && !f16_range_ok(*guard) ? S_alt : S;
}
// The sum of S partial sums at float4 v.  Added in fp64: with up to 64 of them the fp32 additions were
// a third of a projection's error.  Four requests go out together: one at a time a sum of 32 waits
// for 32 trips to L2.
__device__ __forceinline__ float4 sum_partials(const float *__restrict__ x, int64_t stride, int S,
                                               int64_t v) {
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < S; s += 4) {
        float4 b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int at = s + u < S ? s + u : S - 1;
            b[u] = reinterpret_cast<const float4 *>(x + (int64_t)at * stride)[v];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool on = s + u < S;
            t[0] += on ? b[u].x : 0.f;
            t[1] += on ? b[u].y : 0.f;
            t[2] += on ? b[u].z : 0.f;
            t[3] += on ? b[u].w : 0.f;
        }
    }
    return make_float4((float)t[0], (float)t[1], (float)t[2], (float)t[3]);
}
// mean: where the mean of what the K payloads decode to goes as well, or nullptr
int launch_sum_quantize(int K, const PartialSums &part, const PtrPack<float *> &sums,
                        int64_t count, int qbits, int group, const PtrPack<uint8_t *> &codes,
                        const PtrPack<float *> &scales, float *mean, hipStream_t st);
int launch_dequant_average(int K, const PtrPack<const uint8_t *> &codes,
                           const PtrPack<const float *> &scales, int64_t count, int qbits,
                           int group, float *mean_out, hipStream_t st);

// ---- quantise-only outer step (k_qround.hip) ------------------------------------------
int launch_quant_round(int64_t numel, int qbits, int group, int K, const PtrPack<const void *> &tl,
                       int tl_dtype, const PtrPack<float *> &ef, float *theta, float *vel, double lr,
                       double mu, bool has_prev, const PtrPack<const uint8_t *> &pcodes,
                       const PtrPack<const float *> &pscales, bool requant,
                       const PtrPack<uint8_t *> &codes, const PtrPack<float *> &scales,
                       hipStream_t st);
int launch_requantize(float *x, int64_t count, int qbits, int group, hipStream_t st);
int launch_ef_update(int K, const PtrPack<float *> &ef, const float *d, int64_t numel,
                     hipStream_t st);

// ---- measurement aid (k_peak.hip) -------------------------------------------------------
int launch_mfma_peak(int workgroups, int iters, int operands, float *out, hipStream_t st);
int launch_traffic_probe(int K, const PtrPack<float *> &ef, const PtrPack<const void *> &tl,
                         bool tl_bf16, float *theta, float *vel, int64_t numel, hipStream_t st);

// ---- rank-r products ------------------------------------------------------------------
// P_k = delta_k * Q_in   (delta m x n, q_in r x n, out r x m)
// The reduction is split where the output alone does not fill the GPU: with `partial` the sums over
// the splits are left to the caller, else they are formed here.
int launch_project_p(int mma, int64_t m, int64_t n, int r, int K,
                     const PtrPack<const float *> &delta, const float *q_in,
                     const PtrPack<float *> &out, void *workspace, PartialSums *partial,
                     hipStream_t st);
// Q_k = delta_k^T * P_hat (p_hat r x m, out r x n); splits as above
int launch_project_q(int mma, int64_t m, int64_t n, int r, int K,
                     const PtrPack<const float *> &delta, const float *p_hat,
                     const PtrPack<float *> &out, void *workspace, PartialSums *partial,
                     hipStream_t st);
// out[k] = sum_s slabs[k][s], s in index order
int launch_sum_slabs(int K, const PartialSums &part, const PtrPack<float *> &outs, int64_t count,
                     hipStream_t st);
// What happens to each tile d of delta_hat = P_hat Q_bar^T, in this order:
//   out            : d is written
//   K > 0          : e_k <- e_k - d                     (error buffers of Alg. 2)
//   tl_on          : e_k <- (theta - theta_l,k) + e_k   (next pseudo-gradient, same buffer)
//   apply          : vel <- mu vel + d ; theta <- theta - lr (d + mu vel)   (OuterOpt)
struct ReconEpilogue {
    float *out;
    int K;
    PtrPack<float *> ef;
    PtrPack<const void *> tl;
    int tl_on, tl_bf16;
    float *theta, *vel;
    int apply;
    float lr, mu;
};
int launch_reconstruct(int mma, int64_t m, int64_t n, int r, const float *p_hat,
                       const float *q_bar, const ReconEpilogue &ep, void *workspace,
                       hipStream_t st);
size_t project_workspace_bytes(int mma, int64_t m, int64_t n, int r, int K);
size_t reconstruct_workspace_bytes(int mma, int64_t m, int64_t n, int r);

// ---- orthonormalisation and effective rank (k_orth.hip, k_rank.hip) ---------------------
__device__ __forceinline__ double read_lane(double x, int lane) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// the value of lane X of the lane's row of 16
template <int X>
__device__ __forceinline__ double row_bcast(double x) {
    const long long u = __double_as_longlong(x);
    return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, u, 0x150 + X, 0xf, 0xf, true));
}
// f(0), f(1), .. f(N - 1) with the index as a compile-time constant
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        unrolled<N, I + 1>(f);
    }
}

// LDS written and read by the same wavefront: its instructions execute in order, so only the
// compiler has to be kept from reordering.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef double f64x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4_t mfma64(double a, double b, f64x4_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Partial sums of the Gram matrix: elements of the long side in each, and of each quarter of one, which a
// wavefront adds up by itself.
constexpr int kGramChunk = 512;
constexpr int kGramQuarter = kGramChunk / 4;
// Sixteen elements of a quarter: lane (row, q) has elements 4 q .. 4 q + 3 of its row, and the s-th of them
// feeds the s-th product, here and in gram_partial_kernel: the bits of a sum hang on that order.
__device__ __forceinline__ f64x4_t gram_step(const float4 &x, f64x4_t acc) {
    acc = mfma64((double)x.x, (double)x.x, acc);
    acc = mfma64((double)x.y, (double)x.y, acc);
    acc = mfma64((double)x.z, (double)x.z, acc);
    return mfma64((double)x.w, (double)x.w, acc);
}

inline size_t a256x(size_t x) { return (x + 255) & ~(size_t)255; }
// One r x L factor and its fp64 scratch; a batch of them is passed to a kernel by value.
constexpr int kMaxBatch = 64;
struct FactorItem {
    float *f;        // the factor (read by the Gram kernel, rewritten by apply_w)
    int64_t L;
    int32_t r, nchunks;
    double *part;    // nchunks x r x r partial Gram sums (upper triangles)
    double *g;       // g[0]: the mark of the orthonormalisation; or the tridiagonal matrix (k_rank.hip)
    double *w;       // r x r: transpose of the inverse factor (orthonormalisation only)
    int32_t *out;    // r' (effective rank only)
};
struct FactorBatch {
    int n;
    FactorItem it[kMaxBatch];
};
size_t orth_workspace_bytes(int64_t L, int r);
void orth_item(FactorItem *it, float *p, int64_t L, int r, void *workspace);
int launch_orthonormalize(int64_t L, int r, float *p_inout, void *workspace, hipStream_t st);
int launch_orthonormalize_batch(const FactorBatch &batch, hipStream_t st);
size_t effrank_workspace_bytes(int64_t L, int r);
void effrank_item(FactorItem *it, const float *q_bar, int64_t L, int r, int32_t *out,
                  void *workspace);
int launch_effective_rank(int64_t L, int r, const float *q_bar, double tau, int32_t *rprime_dev,
                          void *workspace, hipStream_t st);
int launch_effective_rank_batch(const FactorBatch &batch, double tau, hipStream_t st);
// fp64 Gram matrix partials of r x L factors: part[chunk][a][b] for a <= b (others untouched)
int gram_chunks(int64_t L);
// (round 1: the second round of the orthonormalisation, which factors may not need; else 0)
int launch_gram_partials_batch(const FactorBatch &batch, FactorBatch *reduced, int round,
                               hipStream_t st);

}  // namespace dlcx
