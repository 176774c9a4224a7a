// Orthonormalisation of the averaged factor P_bar (L x r, stored r x L): the thin-QR Q-factor
// with positive diagonal of R, as CholeskyQR with all small-matrix work in fp64:
//   1. G = P^T P as fp64 partial sums over chunks of L (fixed chunking, summed in chunk order)
//   2. one workgroup: scale G to unit diagonal, Cholesky G = R^T R, W = R^-1  (r x r, fp64)
//   3. P <- P W, in place, fp64 accumulation
// Scaling the columns of P does not change the Q-factor, and makes the Cholesky factorisation
// insensitive to the very different column norms a warm-started basis produces.  A pivot of the
// scaled matrix is (residual norm / column norm)^2, so the rule "residual <= 1e-6 of the column
// norm => zero column" is a comparison of the pivot with 1e-12.
//
// The three steps run twice when the first round may have left an orthogonality error that shows
// in fp32: that error is of the order of eps64 ||R^-1||^2, and step 2 has R^-1 at hand, so it
// leaves a mark (kDone) beside its scratch and the kernels of the second round return at once.
//
// All three steps are contractions in fp64 and run on v_mfma_f64_16x16x4_f64.  Its operands, for
// lane l: A[l % 16][l / 16], B[l / 16][l % 16], D[4 v + l / 16][l % 16] in register v.  An operand
// that is already an accumulator (a 16 x 16 block X in D's layout) is, register by register, the
// B operand X and the A operand X^T of a product over its rows.
//
// Every kernel here takes a batch of factors (one descriptor per matrix, passed by value): the
// work per matrix is small and latency-bound, so the matrices of a stage go through each step
// together, one workgroup (or one slice of the grid) per matrix.  What a factor's result is made of
// does not depend on the batch it comes in, but for the rounding of the norm behind the mark (added
// up per wavefront, of which there are as many as the largest rank of the batch asks for): whether the
// second round runs is the batch's where that norm is within rounding of kOneRoundNorm.
#include "common.h"

namespace dlcx {

constexpr int kGramChunk = 512;  // elements of L per partial sum
constexpr int kGT = 256;

typedef double f64x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4_t mfma64(double a, double b, f64x4_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// it.g[0] after the first round's step 2: a second round would change nothing that fp32 shows
// (||R^-1||_F^2 of the unit-diagonal Gram matrix up to which that holds).  Measured against a 64-bit
// QR at 512 x 8 .. 28672 x 256 and condition numbers 1 .. 1e5: up to 8e7 one round alone is as
// close as two (2.5e-8, the rounding to fp32), at 1e9 it is at 3 - 7e-8; the line leaves a factor of 20.
constexpr double kDone = 1.0;
constexpr double kOneRoundNorm = 4e6;
constexpr int kOdd = 1;  // it.g[kOdd]: the first column that is not finite, as a double (r: none)
__device__ __forceinline__ bool second_round_idle(const FactorItem &it, int round) {
    return round == 1 && it.g[0] == kDone;
}

int gram_chunks(int64_t L) { return (int)ceil_div(L, kGramChunk); }

// part[chunk][a][b] = sum_{i in chunk} f[a][i] * f[b][i] for the tile (ta, tb) of 16 NB x 16 NB
// outputs, ta <= tb.  Each wavefront takes a quarter of the chunk and keeps the whole tile; lane
// (row, q) loads the four consecutive elements 4 q .. 4 q + 3 of its row and feeds element s to
// the s-th product (both operands agree on that order of the reduction index), so operands come
// straight from memory, 64 consecutive bytes per row, and nothing waits at a barrier until the
// four quarters are added in order at the end.
// Bound by the fp64 matrix cores at high rank: seven factors of a 100B-class layer at r = 256
// (77824 rows, 5.1 GFLOP over the upper triangle) take 117 us; through LDS tiles and vector
// fp64 FMAs it was 200 us, and 40 us for a single 512 x 8 factor (64 barriers in a row), now 5.
template <int NB>
__global__ __launch_bounds__(kGT) void gram_partial_kernel(FactorBatch batch, int round) {
    __shared__ double red[4][NB * NB * 4][64];
    const FactorItem it = batch.it[blockIdx.z];
    const int r = it.r;
    const int nt = (r + 16 * NB - 1) / (16 * NB);
    if ((int)blockIdx.x >= it.nchunks || (int)blockIdx.y >= nt * (nt + 1) / 2) return;
    if (second_round_idle(it, round)) return;
    const float *__restrict__ f = it.f;
    const int64_t L = it.L;
    // tile index -> (ta, tb) with ta <= tb
    int t = blockIdx.y, ta = 0;
    while (t >= nt - ta) {
        t -= nt - ta;
        ++ta;
    }
    const int tb = ta + t;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, q = lane >> 4;
    const float *pa[NB], *pb[NB];
#pragma unroll
    for (int x = 0; x < NB; ++x) {  // rows past r: any valid row, their outputs are not stored
        const int a = (ta * NB + x) * 16 + row, b = (tb * NB + x) * 16 + row;
        pa[x] = f + (int64_t)(a < r ? a : r - 1) * L + 4 * q;
        pb[x] = f + (int64_t)(b < r ? b : r - 1) * L + 4 * q;
    }
    constexpr int kQuarter = kGramChunk / 4;
    const int64_t begin = (int64_t)blockIdx.x * kGramChunk + wave * kQuarter;
    int64_t end = begin + kQuarter;
    if (end > L) end = L;  // L is a multiple of 16: a step of 16 is whole or not there
    f64x4_t acc[NB][NB];
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y) acc[x][y] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    if (begin < end) {
        float4 va[NB], vb[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            va[x] = *reinterpret_cast<const float4 *>(pa[x] + begin);
            vb[x] = *reinterpret_cast<const float4 *>(pb[x] + begin);
        }
        for (int64_t i = begin; i < end; i += 16) {
            const int64_t nx = i + 16 < end ? i + 16 : begin;
            float4 na[NB], nb[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                na[x] = *reinterpret_cast<const float4 *>(pa[x] + nx);
                nb[x] = *reinterpret_cast<const float4 *>(pb[x] + nx);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
#pragma unroll
                for (int x = 0; x < NB; ++x)
#pragma unroll
                    for (int y = 0; y < NB; ++y) {
                        if (x > y && ta == tb) continue;  // below the diagonal
                        const float fa = s == 0 ? va[x].x : s == 1 ? va[x].y : s == 2 ? va[x].z : va[x].w;
                        const float fb = s == 0 ? vb[y].x : s == 1 ? vb[y].y : s == 2 ? vb[y].z : vb[y].w;
                        acc[x][y] = mfma64((double)fa, (double)fb, acc[x][y]);
                    }
            }
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                va[x] = na[x];
                vb[x] = nb[x];
            }
        }
    }
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][(x * NB + y) * 4 + v][lane] = acc[x][y][v];
    __syncthreads();
    double *dst = it.part + (int64_t)blockIdx.x * r * r;
#pragma unroll
    for (int u = 0; u < NB * NB; ++u) {  // a quarter of the tile each, quarters of the chunk in order
        const int e = wave * NB * NB + u;
        const int x = e / (4 * NB), y = (e / 4) % NB, v = e % 4;
        const int a = (ta * NB + x) * 16 + 4 * v + q, b = (tb * NB + y) * 16 + row;
        const double s = ((red[0][e][lane] + red[1][e][lane]) + red[2][e][lane]) + red[3][e][lane];
        if (a < r && b < r && a <= b) dst[a * r + b] = s;
    }
}

// part[0][a][b] <- sum over the chunks, in chunk order, for a <= b: the sum that the one workgroup
// per matrix of the Cholesky and eigenvalue kernels would otherwise form by itself, here spread
// over the GPU.  Same additions in the same order, so the same bits.  Eight chunks are requested
// before the first is added.
__global__ __launch_bounds__(kGT) void gram_reduce_kernel(FactorBatch batch, int round) {
    const FactorItem it = batch.it[blockIdx.y];
    const int r = it.r;
    const int64_t rr = (int64_t)r * r;
    const int64_t x = (int64_t)blockIdx.x * kGT + threadIdx.x;
    if (x >= rr || it.nchunks < 2) return;
    if (x / r > x % r) return;  // lower triangle: never written, never read
    if (second_round_idle(it, round)) return;
    double s = 0.0;
    int c = 0;
    for (; c + 8 <= it.nchunks; c += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = it.part[(int64_t)(c + u) * rr + x];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; c < it.nchunks; ++c) s += it.part[(int64_t)c * rr + x];
    it.part[x] = s;
}

// Largest rank of a batch for which the consumers add up chunks themselves.
constexpr int kSumRank = 144;

// Partial Gram sums of every factor of the batch, then their sum in part[0]: *reduced is the
// batch as the kernels that consume the Gram matrices have to see it (one chunk each).  Small
// sums are left to the consumer: a launch costs more than the few loads per entry it saves.
int launch_gram_partials_batch(const FactorBatch &batch, FactorBatch *reduced, int round,
                               hipStream_t st) {
    int max_chunks = 1, max_r = 1;
    int64_t max_sum = 1;
    for (int i = 0; i < batch.n; ++i) {
        const int r = batch.it[i].r;
        const int64_t sum = (int64_t)batch.it[i].nchunks * r * r;
        if (batch.it[i].nchunks > max_chunks) max_chunks = batch.it[i].nchunks;
        if (r > max_r) max_r = r;
        if (sum > max_sum) max_sum = sum;
    }
    const int nb = max_r <= 16 ? 1 : 2;  // 16 x 16 blocks per side of a tile
    const int nt = (max_r + 16 * nb - 1) / (16 * nb);
    const dim3 grid((unsigned)max_chunks, (unsigned)(nt * (nt + 1) / 2), (unsigned)batch.n);
    Timed timed(KID_GRAM, st);
    if (nb == 1)
        hipLaunchKernelGGL(gram_partial_kernel<1>, grid, dim3(kGT), 0, st, batch, round);
    else
        hipLaunchKernelGGL(gram_partial_kernel<2>, grid, dim3(kGT), 0, st, batch, round);
    int rc = check_launch("gram_partials");
    if (rc != DLCX_OK) return rc;
    *reduced = batch;
    if (max_chunks < 2 || (max_r <= kSumRank && max_chunks <= 16 && max_sum <= 16 * 1024)) return DLCX_OK;
    const dim3 rgrid((unsigned)ceil_div((int64_t)max_r * max_r, kGT), (unsigned)batch.n);
    hipLaunchKernelGGL(gram_reduce_kernel, rgrid, dim3(kGT), 0, st, batch, round);
    for (int i = 0; i < batch.n; ++i) reduced->it[i].nchunks = 1;
    return check_launch("gram_reduce");
}

// ---------------------------------------------------------------------------------------------
// W = R^-1 of the scaled Gram matrix, one workgroup per matrix, the matrix in registers.
// G is cut into 16 x 16 blocks; only the blocks (I, J), J <= I, exist, one accumulator each, dealt
// to the wavefronts.  Eliminating [G | 1] block row by block row turns G into R and 1 into
// R^-T = L^-1 (G = L L^T); a block (I, J) holds the rest of G (transposed: rows J, columns I)
// until step J, and from then on block (I, J) of L^-1 under construction, which is final after
// step I.  Step k:
//   V = L_kk^-1 of the block (k, k), by one wavefront (factor_block);
//   panel: block (I, k) -> V G_kI =: X_I (a block of R), block (k, J) -> V (k, J) =: X_J (final);
//          both products take V as A operand and the accumulator as it is as B operand;
//   every block with I > k:  J > k: -= X_J^T X_I ;  J <= k: -= X_I^T X_J  (X_k = V),
//          operands from LDS in accumulator layout, no transposition anywhere.
// The wavefront that owns block (k + 1, k + 1) updates it first and factors it while the others
// are still updating.  r^3 2/3 fp64 operations on one compute unit's matrix cores: r = 256 takes
// 151 us and r = 32 13 us (row by row with the matrix in L2 / LDS: 2530 and 49 us).
// ---------------------------------------------------------------------------------------------
constexpr int kMaxBlocks = DLCX_MAX_RANK / 16;
constexpr int kVPitch = 17;
constexpr int kCT = 512;  // at most 8 wavefronts: 17 blocks each at r = 256, 136 of 256 registers

__device__ __forceinline__ double read_lane(double x, int lane) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// LDS written and read by the same wavefront: its instructions execute in order, so only the
// compiler has to be kept from reordering.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// V = L^-1 of a symmetric 16 x 16 block G = L L^T (pitch kVPitch) by one wavefront: lane c < 16
// holds column c of G, lane 16 + c column c of the unit matrix, and the elimination of row j is a
// product of every column with a scalar read from lane i of row j (G is symmetric).  The square
// roots are left to the end, so the chain from pivot to pivot is a reciprocal and two FMAs.
// Dead pivots (<= 1e-12, or not a number) eliminate nothing and leave a zero row of V.  Returns
// whether one of the first `live` pivots was dead.
__device__ __forceinline__ bool factor_block(const double *g, double *v, int lane, int live) {
    double c[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
        c[i] = lane < 16 ? g[i * kVPitch + lane] : (lane == 16 + i ? 1.0 : 0.0);
    double own = 0.0;  // lane i < 16: pivot i
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const double p = read_lane(c[j], j);
        if (lane == j) own = p;
        const bool dead = !(p > 1e-12);
        double rp = __builtin_amdgcn_rcp(p);
        rp = fma(fma(-p, rp, 1.0), rp, rp);
        rp = fma(fma(-p, rp, 1.0), rp, rp);
        const double t = dead ? 0.0 : c[j] * rp;
#pragma unroll
        for (int i = j + 1; i < 16; ++i) c[i] = fma(-read_lane(c[j], i), t, c[i]);
    }
    const bool dead = !(own > 1e-12);
    const double rs = dead ? 0.0 : 1.0 / sqrt(own);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const double x = c[i] * read_lane(rs, i);
        if (lane >= 16 && lane < 32) v[i * kVPitch + lane - 16] = x;
    }
    return __ballot(dead && lane < 16 && lane < live) != 0;
}

template <int SLOTS>
__global__ __launch_bounds__(kCT) void chol_inverse_kernel(FactorBatch batch, int round) {
    const FactorItem it = batch.it[blockIdx.x];
    if (second_round_idle(it, round)) return;
    const int r = it.r, nchunks = it.nchunks;
    const double *__restrict__ part = it.part;
    double *__restrict__ w = it.w;
    __shared__ double dscale[DLCX_MAX_RANK];  // 1 / column norm (0 for a zero column)
    __shared__ double panel[kMaxBlocks][4][64];
    __shared__ double vbuf[2][16 * kVPitch];
    __shared__ double diag[16 * kVPitch];
    __shared__ double red[kCT / 64];
    __shared__ int any_dead;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int g = lane >> 4, col = lane & 15;
    const int nb = (r + 15) >> 4, nblk = nb * (nb + 1) / 2;
    const int64_t rr = (int64_t)r * r;
    if (tid == 0) any_dead = 0;
    f64x4_t t[SLOTS];
    int id[SLOTS];  // I << 8 | J; past the last block I = 0xff... < 0, which no step asks for
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int b = wave + nw * s;
        int I = 0;
        while ((I + 1) * (I + 2) / 2 <= b) ++I;
        id[s] = b < nblk ? I << 8 | (b - I * (I + 1) / 2) : -1;
    }
    auto load = [&](int s, int v, int q) {  // this lane's element of partial sum q
        const int x = 16 * (id[s] & 0xff) + 4 * v + g, y = 16 * (id[s] >> 8) + col;
        const bool in = id[s] >= 0 && x < r && y < r;  // the upper triangle is what is stored
        const double e = part[q * rr + (in ? (x < y ? x * r + y : y * r + x) : 0)];
        return in ? e : 0.0;
    };
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) t[s][v] = load(s, v, 0);
    // chunk by chunk in order; with few blocks four chunks are requested before the first is added
    constexpr int N = SLOTS <= 2 ? 4 : 1;
    for (int q = 1; SLOTS <= 6 && q < nchunks; q += N) {  // above there is one: kSumRank
        double x[N][SLOTS][4];
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
#pragma unroll
                for (int v = 0; v < 4; ++v) x[u][s][v] = load(s, v, q + u < nchunks ? q + u : q);
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
#pragma unroll
                for (int v = 0; v < 4; ++v) t[s][v] += q + u < nchunks ? x[u][s][v] : 0.0;
    }
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
        if (id[s] >= 0 && (id[s] >> 8) == (id[s] & 0xff))
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * v + g == col) {
                    const double d = t[s][v];
                    dscale[16 * (id[s] & 0xff) + col] = !(d < __builtin_inf()) ? -1.0 : d > 0.0 ? 1.0 / sqrt(d) : 0.0;
                }
    __syncthreads();
    // The first column that is not finite (kOdd).  It and those after it come out as NaN, and must not
    // reach those before it: their rows are zeros here, their columns of W NaN, and apply_w reads zeros
    // for them.  (A product with a zero keeps a NaN: whole blocks of the matrix cores' operands would
    // carry it.)
    int odd = r;
    for (int q = 0; q < r; q += 64) {
        const uint64_t m = __ballot(q + lane < r && dscale[q + lane < r ? q + lane : 0] < 0.0);
        if (m && odd == r) odd = q + __builtin_ctzll(m);
    }
    if (tid == 0) it.g[kOdd] = (double)odd;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        if (id[s] < 0) continue;
        const int I = id[s] >> 8, J = id[s] & 0xff;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double scaled = t[s][v] * (dscale[16 * J + 4 * v + g] * dscale[16 * I + col]);
            t[s][v] = 16 * I + col < odd && 16 * J + 4 * v + g < odd ? scaled : 0.0;
        }
        if (I == 0) {  // block (0, 0)
#pragma unroll
            for (int v = 0; v < 4; ++v) diag[(4 * v + g) * kVPitch + col] = t[s][v];
        }
    }
    // The slot's block, opaque to the compiler at every use: addresses derived from it would
    // otherwise be kept for all slots across the loop, and the blocks spilled for them.
    auto block_of = [&](int s, int &I, int &J) {
        int x = id[s];
        asm volatile("" : "+s"(x));
        I = x >> 8;
        J = x & 0xff;
    };
    auto w_entry = [&](int row, int c, double x) {
        return c >= odd ? __builtin_nan("") : row < odd ? dscale[row] * x : 0.0;
    };
    bool dead = false;
    double norm2 = 0.0;  // this lane's share of ||R^-1||_F^2 (of the scaled matrix)
    if (wave == 0) {
        wave_sync();
        dead = factor_block(diag, vbuf[0], lane, r);
    }
    __syncthreads();
    for (int k = 0; k < nb; ++k) {
        const double *vk = vbuf[k & 1];
        double va[4];  // V as A operand
#pragma unroll
        for (int s = 0; s < 4; ++s) va[s] = vk[col * kVPitch + 4 * s + g];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            int I, J;
            block_of(s, I, J);
            if ((I == k) != (J == k) && (I == k || J == k)) {
                f64x4_t x = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int q = 0; q < 4; ++q) x = mfma64(va[q], t[s][q], x);
                const int other = I == k ? J : I;
#pragma unroll
                for (int v = 0; v < 4; ++v) panel[other][v][lane] = x[v];
                if (I == k) {  // a final block of L^-1: W is its transpose, columns scaled
                    t[s] = x;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        norm2 = fma(x[v], x[v], norm2);
                        const int c = 16 * k + 4 * v + g, kk = 16 * J + col;
                        if (c < r) w[(int64_t)kk * r + c] = w_entry(kk, c, x[v]);
                    }
                } else {
                    t[s] = f64x4_t{0.0, 0.0, 0.0, 0.0};
                }
            } else if (I == k) {  // (k, k): V itself
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double x = vk[(4 * v + g) * kVPitch + col];
                    panel[k][v][lane] = x;
                    norm2 = fma(x, x, norm2);
                    const int c = 16 * k + 4 * v + g, kk = 16 * k + col;
                    if (c < r && kk < r) w[(int64_t)kk * r + c] = w_entry(kk, c, x);
                }
            }
        }
        __syncthreads();
        if (k + 1 == nb) break;
        auto update = [&](f64x4_t &acc, int I, int J) {
            const int a = J > k ? J : I, b = J > k ? I : J;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = mfma64(-panel[a][q][lane], panel[b][q][lane], acc);
        };
        bool owner = false;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
            if (id[s] == ((k + 1) << 8 | (k + 1))) {
                update(t[s], k + 1, k + 1);
#pragma unroll
                for (int v = 0; v < 4; ++v) diag[(4 * v + g) * kVPitch + col] = t[s][v];
                owner = true;
            }
        if (owner) {
            wave_sync();
            dead |= factor_block(diag, vbuf[(k + 1) & 1], lane, r - 16 * (k + 1));
        }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            int I, J;
            block_of(s, I, J);
            if (I > k && !(I == k + 1 && J == k + 1)) update(t[s], I, J);
        }
        __syncthreads();
    }
    if (round != 0) return;
    // The orthogonality error of P W is about eps64 ||R^-1||^2 (the Gram sums are good to a few
    // eps64 of the unit diagonal); a factor with a dead column always takes the second round.
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) norm2 += __shfl_xor(norm2, off, 64);
    if (lane == 0) {
        red[wave] = norm2;
        if (dead) any_dead = 1;
    }
    __syncthreads();
    if (tid == 0) {
        double sum = 0.0;
        for (int q = 0; q < nw; ++q) sum += red[q];
        it.g[0] = any_dead == 0 && sum <= kOneRoundNorm ? kDone : 0.0;
    }
}

// P <- P W in place, fp64 accumulation.  Workgroup: 64 consecutive elements of every factor column,
// staged in LDS in fp32 (they are all read before the first is overwritten).  W is upper
// triangular; a wavefront produces 16 columns at a time over the 64 elements: A = W^T (one double
// per lane and step, 16 consecutive columns of four rows, straight from L2, four steps ahead),
// B = P from LDS (16 bytes per lane: lane n holds elements 4 n .. 4 n + 3, element q feeds product
// q), so one element of W serves four products.  The column blocks are dealt so that every
// wavefront gets long and short ones.
// Bound by the fp64 matrix cores: seven factors of a 100B-class layer at r = 256 (77824 rows,
// 5.1 GFLOP) take 130 us (vector fp64 FMAs with W through LDS: 598 us).
__global__ __launch_bounds__(kGT) void apply_w_kernel(FactorBatch batch, int round) {
    extern __shared__ __attribute__((aligned(16))) float fl[];  // [16 nb][64]
    const FactorItem it = batch.it[blockIdx.y];
    const int64_t L = it.L;
    const int64_t i0 = (int64_t)blockIdx.x * 64;
    if (i0 >= L) return;
    if (second_round_idle(it, round)) return;
    float *__restrict__ p = it.f;
    const double *__restrict__ w = it.w;
    const int r = it.r, nb = (r + 15) >> 4, odd = __builtin_amdgcn_readfirstlane((int)it.g[kOdd]);
    for (int idx = threadIdx.x; idx < nb * 256; idx += kGT) {
        const int c = idx >> 4, c4 = idx & 15;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c < odd && i0 + c4 * 4 < L)  // odd <= r
            v = *reinterpret_cast<const float4 *>(p + (int64_t)c * L + i0 + c4 * 4);
        *reinterpret_cast<float4 *>(fl + c * 64 + c4 * 4) = v;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    for (int u = 0; 4 * u < nb; ++u) {
        // blocks w, 7 - w, 8 + w, 15 - w: the work of a block grows with its index
        const int cb = 4 * u + ((u & 1) ? 3 - wave : wave);
        if (cb >= nb) continue;
        const int c = cb * 16 + n;  // A: column of W (any valid one past r, not stored)
        const double *wc = w + (c < r ? c : r - 1);
        auto load_w = [&](double (&dst)[4], int kb) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = kb * 16 + 4 * s + g;
                dst[s] = wc[(int64_t)(k < r ? k : r - 1) * r];
            }
        };
        f64x4_t acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f64x4_t{0.0, 0.0, 0.0, 0.0};
        double a[4];
        load_w(a, 0);
        for (int kb = 0; kb <= cb; ++kb) {
            double an[4];
            load_w(an, kb < cb ? kb + 1 : cb);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float4 b = *reinterpret_cast<const float4 *>(fl + (kb * 16 + 4 * s + g) * 64 + n * 4);
                acc[0] = mfma64(a[s], (double)b.x, acc[0]);
                acc[1] = mfma64(a[s], (double)b.y, acc[1]);
                acc[2] = mfma64(a[s], (double)b.z, acc[2]);
                acc[3] = mfma64(a[s], (double)b.w, acc[3]);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) a[s] = an[s];
        }
        if (i0 + n * 4 < L) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int oc = cb * 16 + 4 * v + g;
                if (oc < r)
                    *reinterpret_cast<float4 *>(p + (int64_t)oc * L + i0 + n * 4) =
                        make_float4((float)acc[0][v], (float)acc[1][v], (float)acc[2][v],
                                    (float)acc[3][v]);
            }
        }
    }
}

size_t orth_workspace_bytes(int64_t L, int r) {
    // partials + g (pitch r + 1) + w
    return a256x(((size_t)gram_chunks(L) * r * r + (size_t)r * (r + 1) + (size_t)r * r) *
                 sizeof(double));
}

static int cholqr_round(const FactorBatch &batch, int round, hipStream_t st) {
    FactorBatch summed;  // the same factors with their Gram sums in one chunk
    int rc = launch_gram_partials_batch(batch, &summed, round, st);
    if (rc != DLCX_OK) return rc;
    int max_nb = 1;
    int64_t max_rows = 1;
    for (int i = 0; i < batch.n; ++i) {
        const int nb = (batch.it[i].r + 15) / 16;
        if (nb > max_nb) max_nb = nb;
        if (ceil_div(batch.it[i].L, 64) > max_rows) max_rows = ceil_div(batch.it[i].L, 64);
    }
    {
        // accumulator blocks per wavefront: 2 up to r = 80, 6 up to r = 144, else 17
        Timed timed(KID_CHOL, st);
        const int blocks = max_nb * (max_nb + 1) / 2, waves = kCT / 64;
        const dim3 grid((unsigned)batch.n), threads((unsigned)(blocks < waves ? blocks : waves) * 64);
        static_assert(6 * 8 >= (kSumRank / 16) * (kSumRank / 16 + 1) / 2, "ranks that sum chunks have at most 6");
        if (blocks <= 2 * waves)
            hipLaunchKernelGGL(chol_inverse_kernel<2>, grid, threads, 0, st, summed, round);
        else if (blocks <= 6 * waves)
            hipLaunchKernelGGL(chol_inverse_kernel<6>, grid, threads, 0, st, summed, round);
        else
            hipLaunchKernelGGL(chol_inverse_kernel<17>, grid, threads, 0, st, summed, round);
        rc = check_launch("chol_inverse");
    }
    if (rc != DLCX_OK) return rc;
    const size_t a_bytes = (size_t)max_nb * 16 * 64 * sizeof(float);
    static size_t apply_granted = 0;
    rc = grant_dynamic_lds(reinterpret_cast<const void *>(apply_w_kernel), a_bytes, &apply_granted,
                       "apply_w attribute");
    if (rc != DLCX_OK) return rc;
    Timed timed(KID_APPLY_W, st);
    hipLaunchKernelGGL(apply_w_kernel, dim3((unsigned)max_rows, (unsigned)batch.n), dim3(kGT),
                       a_bytes, st, batch, round);
    return check_launch("apply_w");
}

// Fills the scratch pointers of item i from a workspace of orth_workspace_bytes(L, r) bytes.
void orth_item(FactorItem *it, float *p, int64_t L, int r, void *workspace) {
    it->f = p;
    it->L = L;
    it->r = r;
    it->nchunks = gram_chunks(L);
    it->part = reinterpret_cast<double *>(workspace);
    it->g = it->part + (size_t)it->nchunks * r * r;
    it->w = it->g + (size_t)r * (r + 1);
    it->out = nullptr;
}

int launch_orthonormalize_batch(const FactorBatch &batch, hipStream_t st) {
    if (batch.n == 0) return DLCX_OK;
    int rc = cholqr_round(batch, 0, st);
    if (rc != DLCX_OK) return rc;
    return cholqr_round(batch, 1, st);
}

int launch_orthonormalize(int64_t L, int r, float *p_inout, void *workspace, hipStream_t st) {
    FactorBatch b;
    b.n = 1;
    orth_item(&b.it[0], p_inout, L, r, workspace);
    return launch_orthonormalize_batch(b, st);
}

}  // namespace dlcx
