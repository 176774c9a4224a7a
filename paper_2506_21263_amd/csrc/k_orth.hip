// Orthonormalisation of the averaged factor P_bar (L x r, stored r x L): the thin-QR Q-factor
// with positive diagonal of R, as CholeskyQR with all small-matrix work in fp64:
//   1. G = P^T P as fp64 partial sums over chunks of L (fixed chunking, summed in chunk order)
//   2. one workgroup: scale G to unit diagonal, Cholesky G = R^T R, W = R^-1  (r x r, fp64, kept as W^T)
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
// does not depend on the batch it comes in, but above rank 16 for the rounding of the norm behind the
// mark (added up per wavefront, of which there are as many as the largest rank of the batch asks
// for): whether the second round runs is the batch's where that norm is within rounding of kOneRoundNorm.
#include <type_traits>

#include "common.h"

namespace dlcx {

constexpr int kGT = 256;

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

// Work of a batch along one grid dimension: item i has the places first[i] .. first[i + 1] - 1.  (A grid as
// long as the longest factor for every item: of a 100B-class layer's seven, one of 28672 rows beside six of
// 8192, three workgroups in five had nothing to do but took their turn, and in apply_w 64 KB of LDS.)
struct Places {
    int first[kMaxBatch + 1];
};
// Items of `each` places, one along y: with nothing to look up before an item's description is read, every
// launch is 0.1 us shorter, a whole orthonormalisation 0.3 - 0.4.
struct Even {
    int each;
};
// A launch has less than 2^32 threads along x: longer rows of chunks (36 tiles of 256 threads each at most) and
// of apply_w's workgroups (512 threads at most) go on along y, as Places.
constexpr int kMostChunks = 1 << 18;
constexpr int kMostRows = 1 << 22;
// The item that `place` of row blockIdx.y belongs to, by every wavefront for itself, or -1; `place` becomes the
// place inside it.  (Past the last item first[] stays at its end, so the number of items is not waited for.)
__device__ __forceinline__ int item_of(const Places &at, int most, int &place) {
    place += blockIdx.y * most;
    static_assert(kMaxBatch == 64, "one lane per item");
    const uint64_t m = __ballot(at.first[threadIdx.x & 63] <= place);
    const int i = __builtin_amdgcn_readfirstlane(__popcll(m) - 1);
    if (place >= at.first[kMaxBatch]) return -1;
    place -= at.first[i];
    return i;
}
__device__ __forceinline__ int item_of(const Even &at, int, int &place) {
    return place < at.each ? (int)blockIdx.y : -1;
}
// launch(places, x, y) for count(item) places of every item, at most `most` along x; several items as Even only
// where theirs are whole granules
template <typename F, typename G>
static int for_places(const FactorBatch &batch, int most, int granule, F &&count, G &&launch) {
    Places at;
    at.first[0] = 0;
    const int64_t each = count(batch.it[0]);
    bool even = each <= most && (batch.n == 1 || each % granule == 0);
    for (int i = 0; i < kMaxBatch; ++i) {
        const int64_t places = i < batch.n ? count(batch.it[i]) : 0;
        at.first[i + 1] = at.first[i] + (int)places;
        even = even && (i >= batch.n || places == each);
    }
    if (even) return launch(Even{(int)each}, (int)each, batch.n);
    const int all = at.first[batch.n];
    return launch(at, all < most ? all : most, (int)ceil_div(all, most));
}

int gram_chunks(int64_t L) { return (int)ceil_div(L, kGramChunk); }

// part[chunk][a][b] = sum_{i in chunk} f[a][i] * f[b][i] for the tile (ta, tb) of 16 NB x 16 NB
// outputs, ta <= tb.  Each wavefront takes a quarter of the chunk and keeps the whole tile; lane
// (row, q) loads the four consecutive elements 4 q .. 4 q + 3 of its row and feeds element s to
// the s-th product (both operands agree on that order of the reduction index), so operands come
// straight from memory, 64 consecutive bytes per row, and nothing waits at a barrier until the
// four quarters are added in order at the end.
// Bound by the fp64 matrix cores at high rank: seven factors of a 100B-class layer at r = 256
// (77824 rows, 5.4 GFLOP over the upper triangle, 69 us at the datasheet's rate) take 110 us (118 with one loop
// for all tiles, whose branch copied accumulators); through LDS tiles and vector fp64 FMAs it was 200 us, and
// 40 us for a single 512 x 8 factor (64 barriers in a row), now 5.
// From kGroupedChunks on, the tiles of a chunk are consecutive workgroups of one XCD (every eighth workgroup of the
// grid), eight chunks side by side: a chunk, 512 KB at r = 256, is read from memory once and 36 times from that
// XCD's L2.  Fewer chunks would leave some XCDs with more of them than others, or with none: their tiles go to
// all XCDs in turn.
constexpr int kGroupedChunks = 64;
template <int NB, typename At>
__global__ __launch_bounds__(kGT, 4) void gram_partial_kernel(FactorBatch batch, At at, int tiles, bool grouped, int round) {
    __shared__ double red[4][NB * NB * 4][64];
    const int slot = grouped ? blockIdx.x >> 3 : blockIdx.x;
    int chunk = slot / tiles, t = slot - chunk * tiles;
    if (grouped) chunk = 8 * chunk + (blockIdx.x & 7);
    const int item = item_of(at, kMostChunks, chunk);
    if (item < 0) return;
    const FactorItem it = batch.it[item];
    const int r = it.r;
    const int nt = (r + 16 * NB - 1) / (16 * NB);
    if (t >= nt * (nt + 1) / 2) return;
    if (second_round_idle(it, round)) return;
    const float *__restrict__ f = it.f;
    const int64_t L = it.L;
    // tile index -> (ta, tb) with ta <= tb
    int ta = 0;
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
    const int64_t begin = (int64_t)chunk * kGramChunk + wave * kGramQuarter;
    int64_t end = begin + kGramQuarter;
    if (end > L) end = L;  // L is a multiple of 16: a step of 16 is whole or not there
    f64x4_t acc[NB][NB];
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y) acc[x][y] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    auto sums = [&](auto diagonal) {
        if (begin >= end) return;
        float4 va[2][NB], vb[2][NB];
        auto load = [&](int set, int64_t i) {
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                va[set][x] = *reinterpret_cast<const float4 *>(pa[x] + i);
                vb[set][x] = *reinterpret_cast<const float4 *>(pb[x] + i);
            }
            __builtin_amdgcn_sched_barrier(0);  // the requests go out before the products they do not belong to
        };
        auto multiply = [&](int set) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int x = 0; x < NB; ++x)
#pragma unroll
                    for (int y = 0; y < NB; ++y) {
                        if (diagonal && x > y) continue;  // below the diagonal
                        const float4 &a = va[set][x], &b = vb[set][y];
                        const float fa = s == 0 ? a.x : s == 1 ? a.y : s == 2 ? a.z : a.w;
                        const float fb = s == 0 ? b.x : s == 1 ? b.y : s == 2 ? b.z : b.w;
                        acc[x][y] = mfma64((double)fa, (double)fb, acc[x][y]);
                    }
            __builtin_amdgcn_sched_barrier(0);
        };
        load(0, begin);
        for (int64_t i = begin; i < end; i += 32) {
            load(1, i + 16 < end ? i + 16 : begin);
            multiply(0);
            if (i + 16 >= end) break;
            load(0, i + 32 < end ? i + 32 : begin);
            multiply(1);
        }
    };
    if (ta == tb) sums(std::true_type());  // two loops: one with a branch in it copied its accumulators about
    else sums(std::false_type());
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < NB; ++y)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][(x * NB + y) * 4 + v][lane] = acc[x][y][v];
    __syncthreads();
    double *dst = it.part + (int64_t)chunk * r * r;
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
    int64_t max_sum = 1, chunks = 0;
    for (int i = 0; i < batch.n; ++i) {
        const int r = batch.it[i].r;
        chunks += batch.it[i].nchunks;
        const int64_t sum = (int64_t)batch.it[i].nchunks * r * r;
        if (batch.it[i].nchunks > max_chunks) max_chunks = batch.it[i].nchunks;
        if (r > max_r) max_r = r;
        if (sum > max_sum) max_sum = sum;
    }
    const int nb = max_r <= 16 ? 1 : 2;  // 16 x 16 blocks per side of a tile
    const int nt = (max_r + 16 * nb - 1) / (16 * nb);
    const int tiles = nt * (nt + 1) / 2;
    const bool grouped = chunks >= kGroupedChunks;
    static_assert(kMostChunks % 8 == 0, "whole groups of eight chunks");
    auto count = [](const FactorItem &it) { return (int64_t)it.nchunks; };
    Timed timed(KID_GRAM, st);
    int rc = for_places(batch, kMostChunks, grouped ? 8 : 1, count, [&](auto at, int x, int y) {
        const dim3 grid((unsigned)(grouped ? ceil_div(x, 8) * 8 : x) * (unsigned)tiles, (unsigned)y);
        using At = decltype(at);
        if (nb == 1)
            hipLaunchKernelGGL((gram_partial_kernel<1, At>), grid, dim3(kGT), 0, st, batch, at, tiles, grouped, round);
        else
            hipLaunchKernelGGL((gram_partial_kernel<2, At>), grid, dim3(kGT), 0, st, batch, at, tiles, grouped, round);
        return check_launch("gram_partials");
    });
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
// G is cut into 16 x 16 blocks; only the blocks (I, J), J <= I, exist, one accumulator each: the last
// wavefront holds those on the diagonal, the others are dealt out.  Eliminating [G | 1] block row by block row
// turns G into R and 1 into R^-T = L^-1 (G = L L^T); a block (I, J) holds the rest of G (transposed: rows J,
// columns I) until step J, and from then on block (I, J) of L^-1 under construction, which is final after
// step I.  Step k, with V = L_kk^-1 of the block (k, k) from the step before:
//   panel: block (I, k) -> V G_kI =: X_I (a block of R), block (k, J) -> V (k, J) =: X_J (final);
//          both products take V as A operand and the accumulator as it is as B operand;
//   every block with I > k:  J > k: -= X_J^T X_I ;  J <= k: -= X_I^T X_J  (X_k = V),
//          operands from LDS in accumulator layout, no transposition anywhere;
//   the diagonal's wavefront updates (k + 1, k + 1) first and factors it while the others are updating.
// r^3 2/3 fp64 operations on one compute unit's matrix cores, 36 us at r = 256 at their rate (64 clocks an
// instruction).  A wavefront runs through its blocks by a mask of those that a step concerns; loads, scaling and
// stores are a handful of instructions a block (70 KB of instructions before, fetched from memory once per launch:
// 22 us to load the matrix); and the wavefront that factors has little else to do, where all waited for its
// other updates.  r = 256 takes 104 us: 16 steps of 5 us, of which the products 3.3, panel and barriers 1.3, and 20
// us around them (151 before; row by row with the matrix in L2: 2530); r = 32 with up to 16 sums 9 us.
// ---------------------------------------------------------------------------------------------
constexpr int kMaxBlocks = DLCX_MAX_RANK / 16;
constexpr int kVPitch = 17;  // of a 16 x 16 block in LDS
constexpr int kCT = 512;  // at most 8 wavefronts: 18 blocks each at r = 256, 144 of 256 registers

// V = L^-1 of a symmetric 16 x 16 block G = L L^T by one wavefront, both as accumulators: register q of
// lane (g, col) = (lane / 16, lane % 16) is element (4 q + g, col).  Eliminating row j from [G | 1] is a product
// with one row of the operands in use, -(row j) / pivot as A (G is symmetric) and row j as B, and row j of an
// accumulator lies where both want row j % 4 of their four: no lane needs another's value but for the pivots.
// The pivot after is worked out beside the product that makes its row, by the same operations.  The square roots
// are left to the end.  Dead pivots (<= 1e-12, or not a number) eliminate nothing and leave a zero row of V.
// Writes V as the A operand of the panel reads it (pitch kVPitch) and as an accumulator; returns whether one
// of the first `live` pivots was dead.
// Bound by the chain from pivot to pivot, 330 clocks each.  (Rows spread over the lanes by permlane and
// updated by vector instructions, 70 of them a pivot: 109 us instead of 104 for the kernel below at r = 256;
// not unrolled, with the registers selected by the row: 125.)
__device__ __forceinline__ bool factor_block(f64x4_t t, double *va, double (*vb)[64], int lane, int live) {
    const int g = lane >> 4, col = lane & 15;
    f64x4_t u, own;  // the right half; the pivot of each row
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = 4 * q + g == col ? 1.0 : 0.0;
    double p = read_lane(t[0], 0);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int q = j / 4, q1 = (j + 1) / 4;
        const bool mine = g == j % 4;
        if (mine) own[q] = p;
        if (j == 15) break;
        double rp = __builtin_amdgcn_rcp(p);
        rp = fma(fma(-p, rp, 1.0), rp, rp);
        rp = fma(fma(-p, rp, 1.0), rp, rp);
        rp = p > 1e-12 ? rp : 0.0;
        const double x = read_lane(t[q], 16 * (j % 4) + j + 1);
        const double d = read_lane(t[q1], 16 * ((j + 1) % 4) + j + 1);
        p = fma(-x * rp, x, d);
        const double row = mine ? t[q] : 0.0;
        const double a = col > j ? -row * rp : 0.0;  // rows that are done keep what they have
        t = mfma64(a, row, t);
        u = mfma64(a, mine ? u[q] : 0.0, u);
    }
    bool any = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool dead = !(own[q] > 1e-12);
        double y = __builtin_amdgcn_rsq(own[q]);
        y = fma(0.5 * y, fma(-own[q] * y, y, 1.0), y);
        y = fma(0.5 * y, fma(-own[q] * y, y, 1.0), y);
        const double x = dead ? 0.0 : u[q] * y;
        va[(4 * q + g) * kVPitch + col] = x;
        vb[q][lane] = x;
        any = any || (dead && 4 * q + g < live);
    }
    return __ballot(any) != 0;
}

// Blocks of a side that SLOTS of every wavefront but the diagonal's have room for.  What a workgroup takes of LDS
// hangs on it: 25 KB up to r = 64, 29 to 80, 45 to 144, else 74.
constexpr int most_blocks(int slots) {
    int nb = 1;
    while (nb < kMaxBlocks && (nb + 1) * nb / 2 <= slots * (kCT / 64 - 1)) ++nb;
    return slots > 6 ? kMaxBlocks : nb;
}

template <int SLOTS>
__global__ __launch_bounds__(kCT) void chol_inverse_kernel(FactorBatch batch, int round) {
    const FactorItem it = batch.it[blockIdx.x];
    if (second_round_idle(it, round)) return;
    const int r = it.r, nchunks = it.nchunks;
    const double *__restrict__ part = it.part;
    double *__restrict__ w = it.w;
    constexpr int kBlocks = most_blocks(SLOTS);  // of a side
    __shared__ double dscale[16 * kBlocks];   // 1 / column norm (0 for a zero column)
    __shared__ double panel[kBlocks][4][64];
    __shared__ double diag[kBlocks][4][64];   // the blocks on the diagonal
    __shared__ double va[2][16 * kVPitch];    // V of even and odd steps, as A operand ..
    __shared__ double vb[2][4][64];           // .. and as accumulator
    __shared__ double red[kCT / 64];
    __shared__ int any_dead;
    __shared__ int factored;  // blocks on the diagonal that are
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int g = lane >> 4, col = lane & 15;
    const int nb = (r + 15) >> 4;
    const int64_t rr = (int64_t)r * r;
    const bool diagonal = wave == nw - 1;
    // Lane s: row and column of the block in slot s, or row -1, column 0: none.  (This factor may have fewer
    // blocks than the launch's largest.)
    // A block each in turn.  With many, `beside`, the wavefront on the SIMD of the diagonal's, is left out every
    // third time: fp64 products hold up the fp64 arithmetic of the other wavefront of a SIMD, so it starts on
    // its updates when the factorisation is done.
    const int beside = SLOTS > 6 ? nw - 5 : -1;
    int bI = -1, bJ = 0;
    if (!diagonal && lane < SLOTS) {
        const int others = nw - 1;
        int b = wave + others * lane;
        if (beside >= 0) b -= lane / 3 + (lane % 3 == 2 && wave > beside ? 1 : 0);
        int I = 1;
        while ((I + 1) * I / 2 <= b) ++I;
        if (b < nb * (nb - 1) / 2 && !(wave == beside && lane % 3 == 2)) {
            bI = I;
            bJ = b - I * (I - 1) / 2;
        }
    }
    auto row_of = [&](int s) { return __builtin_amdgcn_readlane(bI, s); };
    auto col_of = [&](int s) { return __builtin_amdgcn_readlane(bJ, s); };
    // All blocks are held negated: what is taken from them is then added.
    f64x4_t t[SLOTS];
    // Where this lane's elements of block (I, J) are in a partial sum.  The upper triangle is what is stored; past
    // the edge the last row or column is read again.
    auto place = [&](int (&at)[4], int I, int J) {
        const int y0 = 16 * I + col, x0 = 16 * J + g, y = y0 < r ? y0 : r - 1;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int x = x0 + 4 * v < r ? x0 + 4 * v : r - 1;
            at[v] = (x < y ? x : y) * r + (x < y ? y : x);
        }
    };
    constexpr int kOnDiagonal = SLOTS <= 2 ? 1 : 2;  // blocks on the diagonal that a wavefront reads: wave, wave + nw
    f64x4_t own[kOnDiagonal];
    auto first = [&](f64x4_t &to, int (&at)[4], int I, int J) {
        place(at, I, J);
#pragma unroll
        for (int v = 0; v < 4; ++v) to[v] = part[at[v]];
        if (SLOTS > 6) __builtin_amdgcn_sched_barrier(0);  // of addresses no more than one block's are in registers
    };
    int at[SLOTS][4], at_own[kOnDiagonal][4];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) first(t[s], at[s], row_of(s) < 0 ? 0 : row_of(s), col_of(s));
#pragma unroll
    for (int s = 0; s < kOnDiagonal; ++s) {
        const int i = wave + nw * s < nb ? wave + nw * s : 0;
        first(own[s], at_own[s], i, i);
    }
    // Chunk by chunk in order; with few blocks three chunks are requested before the first is added.  Of what is
    // requested and not there nothing is added, but it takes as long: with five, 2048 x 64 37.1 us and 8192 x 32
    // 29.3, with three 35.3 and 28.2, the whole orthonormalisation.
    constexpr int N = SLOTS <= 2 ? 3 : 1;
    for (int q = 1; SLOTS <= 6 && q < nchunks; q += N) {  // above there is one: kSumRank
        f64x4_t x[N][SLOTS], y[N][kOnDiagonal];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const double *src = part + (q + u < nchunks ? q + u : q) * rr;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) x[u][s][v] = src[at[s][v]];
#pragma unroll
                for (int s = 0; s < kOnDiagonal; ++s) y[u][s][v] = src[at_own[s][v]];
            }
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const bool on = q + u < nchunks;
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) t[s][v] += on ? x[u][s][v] : 0.0;
#pragma unroll
                for (int s = 0; s < kOnDiagonal; ++s) own[s][v] += on ? y[u][s][v] : 0.0;
            }
    }
    if (tid == 0) {
        any_dead = 0;
        factored = 0;
    }
#pragma unroll
    for (int s = 0; s < kOnDiagonal; ++s) {
        const int i = wave + nw * s;
        if (i >= nb) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (4 * v + g == col) dscale[16 * i + col] = own[s][v];
    }
    __syncthreads();
    for (int q = tid; q < 16 * nb; q += blockDim.x) {
        const double d = dscale[q];
        dscale[q] = q >= r ? 0.0 : !(d < __builtin_inf()) ? -1.0 : d > 0.0 ? 1.0 / sqrt(d) : 0.0;
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
    auto scale = [&](f64x4_t &x, int I, int J) {
        const double dc = -dscale[16 * I + col];
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] *= dscale[16 * J + 4 * v + g] * dc;
        if (odd < r)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = 16 * I + col < odd && 16 * J + 4 * v + g < odd ? x[v] : 0.0;
    };
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) scale(t[s], row_of(s) < 0 ? 0 : row_of(s), col_of(s));
#pragma unroll
    for (int s = 0; s < kOnDiagonal; ++s) {
        const int i = wave + nw * s;
        if (i >= nb) continue;
        scale(own[s], i, i);
#pragma unroll
        for (int v = 0; v < 4; ++v) diag[i][v][lane] = own[s][v];
    }
    __syncthreads();
    double norm2 = 0.0;  // this lane's share of ||R^-1||_F^2 (of the scaled matrix)
    // Block (I, J) of L^-1, columns scaled: W^T, whose rows it stores (W itself went out in single numbers, each
    // to a line of its own: 8 - 13 us at r = 256).
    auto store = [&](int I, int J, const f64x4_t &x) {
        const int row = 16 * J + col;
        const double by = row < odd ? dscale[row] : 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = 16 * I + 4 * v + g;
            norm2 = fma(x[v], x[v], norm2);
            if (c < r && row < r) w[c * r + row] = c >= odd ? __builtin_nan("") : by * x[v];
        }
    };
    bool dead = false;
    for (int k = 0; k < nb; ++k) {
        const double (*vk)[64] = vb[k & 1];
        // acc (negated) += the product of its operands X_J and X_I (J > k), or X_I and X_J, of step k - 1
        auto update = [&](f64x4_t &acc, int I, int J, int k, const double (*v)[64]) {
            const double (*pa)[64] = panel[J > k ? J : I];
            const double (*pb)[64] = J > k ? panel[I] : J == k ? v : panel[J];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = mfma64(pa[q][lane], pb[q][lane], acc);
        };
        auto update_diag = [&](int s, int k) {
            f64x4_t x;
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = diag[s][v][lane];
            if (k >= 0) update(x, s, s, k, nullptr);
            return x;
        };
        if (diagonal) {  // the others wait for this wavefront
            __builtin_amdgcn_s_setprio(3);
            dead |= factor_block(-update_diag(k, k - 1), va[k & 1], vb[k & 1], lane, r - 16 * k);
            if (lane == 0) __hip_atomic_store(&factored, k + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (k > 0)
                for (int s = k + 1; s < nb; ++s) {
                    const f64x4_t x = update_diag(s, k - 1);
#pragma unroll
                    for (int v = 0; v < 4; ++v) diag[s][v][lane] = x[v];
                }
            __builtin_amdgcn_s_setprio(0);
        } else if (k > 0) {
            if (wave == beside)  // a matter of speed only: what is read is there since the last barrier
                while (__hip_atomic_load(&factored, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= k)
                    __builtin_amdgcn_s_sleep(1);
            const uint64_t mine = __ballot(bI >= k);
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (mine >> s & 1) update(t[s], row_of(s), col_of(s), k - 1, vb[(k - 1) & 1]);
        }
        __syncthreads();
        if (diagonal) {
            f64x4_t x;
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = vk[v][lane];
            store(k, k, x);
        } else {
            double a[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = -va[k & 1][col * kVPitch + 4 * q + g];
            const uint64_t mine = __ballot(bI == k || (bI > k && bJ == k));
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (mine >> s & 1) {
                    f64x4_t x = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int q = 0; q < 4; ++q) x = mfma64(a[q], t[s][q], x);
                    const int I = row_of(s);
                    double (*to)[64] = panel[I == k ? col_of(s) : I];
#pragma unroll
                    for (int v = 0; v < 4; ++v) to[v][lane] = x[v];
                    t[s] = I == k ? x : f64x4_t{0.0, 0.0, 0.0, 0.0};  // (k, J): a final block of L^-1
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        if (row_of(s) >= 0) store(row_of(s), col_of(s), t[s]);
        __builtin_amdgcn_sched_barrier(0);
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
// triangular; a wavefront produces 16 columns at a time over the 64 elements: A = W^T (four doubles
// per lane and 16 rows of W, consecutive in W^T, straight from L2 a step ahead; the s-th of them feeds the s-th
// product, and B agrees on that order of the reduction index), B = P from LDS (16 bytes per lane: lane n holds
// elements 4 n .. 4 n + 3, element q feeds product q), so one element of W serves four products.  The column blocks are dealt so that every
// wavefront gets long and short ones.
// Bound by the fp64 matrix cores: seven factors of a 100B-class layer at r = 256 (77824 rows,
// 5.4 GFLOP) take 112 us (four wavefronts and a workgroup for every 64 rows of the longest factor: 133; vector
// fp64 FMAs with W through LDS: 598 us).
template <int NW, typename At>  // wavefronts
__global__ __launch_bounds__(64 * NW, 2) void apply_w_kernel(FactorBatch batch, At at, int round) {
    extern __shared__ __attribute__((aligned(16))) float fl[];  // [16 nb][64]
    int place = blockIdx.x;
    const int item = item_of(at, kMostRows, place);
    if (item < 0) return;
    const FactorItem it = batch.it[item];
    const int64_t L = it.L;
    const int64_t i0 = (int64_t)place * 64;
    if (second_round_idle(it, round)) return;
    float *__restrict__ p = it.f;
    const double *__restrict__ w = it.w;
    const int r = it.r, nb = (r + 15) >> 4, odd = __builtin_amdgcn_readfirstlane((int)it.g[kOdd]);
    for (int idx = threadIdx.x; idx < nb * 256; idx += 64 * NW) {
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
    for (int u = 0; NW * u < nb; ++u) {
        // blocks w, 2 NW - 1 - w, 2 NW + w, ..: the work of a block grows with its index
        const int cb = NW * u + ((u & 1) ? NW - 1 - wave : wave);
        if (cb >= nb) continue;
        const int c = cb * 16 + n;  // A: column of W (any valid one past r, not stored)
        const double *wc = w + (int64_t)(c < r ? c : r - 1) * r + 4 * g;
        auto load_w = [&](double (&dst)[4], int kb) {
#pragma unroll
            for (int s = 0; s < 4; ++s) dst[s] = wc[kb * 16 + s];
        };
        f64x4_t acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f64x4_t{0.0, 0.0, 0.0, 0.0};
        auto multiply = [&](const double (&a)[4], int kb) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float4 b = *reinterpret_cast<const float4 *>(fl + (kb * 16 + 4 * g + s) * 64 + n * 4);
                acc[0] = mfma64(a[s], (double)b.x, acc[0]);
                acc[1] = mfma64(a[s], (double)b.y, acc[1]);
                acc[2] = mfma64(a[s], (double)b.z, acc[2]);
                acc[3] = mfma64(a[s], (double)b.w, acc[3]);
            }
        };
        double a[4], last[4];
        if (cb > 0) load_w(a, 0);
#pragma unroll
        for (int s = 0; s < 4; ++s) {  // the block on the diagonal: rows past r are not there
            const int k = cb * 16 + 4 * g + s;
            last[s] = k < r ? wc[cb * 16 + s] : 0.0;
        }
        for (int kb = 0; kb < cb; ++kb) {
            double an[4];
            load_w(an, kb + 1 < cb ? kb + 1 : kb);
            multiply(a, kb);
#pragma unroll
            for (int s = 0; s < 4; ++s) a[s] = an[s];
        }
        multiply(last, cb);
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

// The whole orthonormalisation of small factors, a workgroup each, which holds its factor in LDS: the sums, the
// factorisation and P W as above for a single block, and the second round where the first asks for one.  All
// sums are in the order of the kernels above, that of the norm behind the mark among them (a single block's is
// one wavefront's there too): a batch takes this form if all of its factors are small, and what a factor's result
// is does not hang on that.
// Bound by latency, one workgroup's.  Instead of a chain of six launches, of which the last three mostly only read
// a mark, us in a graph, one launch | six: 512 x 8 8.4 | 16.3, 512 x 16 9.4 | 16.5, 1024 x 16 13.4 | 17.4, 1536 x 8
// 15.2 | 16.8, 1520 x 16 17.5 | 17.5, 2048 x 8 18.4 | 17.2, 2032 x 12 20.5 | 17.3, seven of them 20.8 | 18.0.  From
// the host, which takes longer for six launches than they run: 512 x 8 10.6 | 24.0, 1520 x 16 17.5 | 23.5, 2048 x
// 8 18.4 | 23.4, 2032 x 12 20.5 | 24.1, hence the limits.
constexpr int kSmallOrthRank = 16;
constexpr int kSmallOrthLength = 2048;
constexpr int kSmallFloats = 24 * 1024;  // with the rows' padding, 96 KB
constexpr int kSmallThreads = 512;
static inline size_t small_bytes(int64_t L, int r) { return (size_t)r * (size_t)(L + 4) * sizeof(float); }
__global__ __launch_bounds__(kSmallThreads) void orth_small_kernel(FactorBatch batch) {
    constexpr int NW = kSmallThreads / 64;
    extern __shared__ __attribute__((aligned(16))) float fl[];  // [r][L + 4]: 16 rows start in 64 banks
    __shared__ double red[kSmallOrthLength / kGramQuarter][4][64];
    __shared__ double dscale[16];
    __shared__ double va[16 * kVPitch], wt[16 * kVPitch], vb[4][64];
    __shared__ int state;  // the first column that is not finite, 16 more: a second round is needed
    const FactorItem it = batch.it[blockIdx.x];
    const int r = it.r, L = (int)it.L, pitch = L + 4, quads = L / 4, quarters = 4 * it.nchunks;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *__restrict__ p = it.f;
    for (int c = wave; c < r; c += NW)
        for (int i = lane; i < quads; i += 64)
            *reinterpret_cast<float4 *>(fl + c * pitch + 4 * i) = reinterpret_cast<const float4 *>(p + (int64_t)c * L)[i];
    for (int round = 0; round < 2; ++round) {
        __syncthreads();
        const float *row = fl + (col < r ? col : r - 1) * pitch + 4 * g;  // rows past r: any valid one
        for (int q = wave; q < quarters; q += NW) {  // quarters of the 512-element sums
            f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
            for (int i = q * kGramQuarter; i < (q + 1) * kGramQuarter && i < L; i += 16) {
                acc = gram_step(*reinterpret_cast<const float4 *>(row + i), acc);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) red[q][v][lane] = acc[v];
        }
        __syncthreads();
        if (wave == 0) {
            f64x4_t x;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                x[v] = 0.0;
                for (int q = 0; q < quarters; q += 4)
                    x[v] += ((red[q][v][lane] + red[q + 1][v][lane]) + red[q + 2][v][lane]) + red[q + 3][v][lane];
                if (4 * v + g == col)
                    dscale[col] = col >= r ? 0.0 : !(x[v] < __builtin_inf()) ? -1.0 : x[v] > 0.0 ? 1.0 / sqrt(x[v]) : 0.0;
            }
            wave_sync();
            const double dc = dscale[col];
            const uint64_t m = __ballot(lane < 16 && dc < 0.0);  // columns that are not finite: as in chol_inverse_kernel
            const int odd = m ? __builtin_ctzll(m) : r;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = col < odd && 4 * v + g < odd ? x[v] * (dscale[4 * v + g] * dc) : 0.0;
            const bool dead = factor_block(x, va, vb, lane, r);
            wave_sync();
            double norm2 = 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double y = vb[v][lane];
                const int c = 4 * v + g;
                norm2 = fma(y, y, norm2);
                wt[c * kVPitch + col] = c >= odd ? __builtin_nan("") : col < odd ? dc * y : 0.0;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) norm2 += __shfl_xor(norm2, off, 64);
            if (lane == 0) state = odd + (dead || !(norm2 <= kOneRoundNorm) ? 32 : 0);
        }
        __syncthreads();
        const int odd = state & 31;
        const bool again = state >= 32;
        double a[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s] = wt[col * kVPitch + 4 * g + s];
        for (int i = 16 * wave; i < L; i += 16 * NW) {  // 16 elements of every column, read before they are written
            f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = 4 * g + s;
                const float x = fl[(k < r ? k : 0) * pitch + i + col];
                acc = mfma64(a[s], k < odd ? (double)x : 0.0, acc);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * v + g < r) fl[(4 * v + g) * pitch + i + col] = (float)acc[v];
        }
        if (!again) break;
    }
    __syncthreads();
    for (int c = wave; c < r; c += NW)
        for (int i = lane; i < quads; i += 64)
            reinterpret_cast<float4 *>(p + (int64_t)c * L)[i] = *reinterpret_cast<const float4 *>(fl + c * pitch + 4 * i);
}

size_t orth_workspace_bytes(int64_t L, int r) {
    // partials + g (pitch r + 1) + w
    return a256x(((size_t)gram_chunks(L) * r * r + (size_t)r * (r + 1) + (size_t)r * r) *
                 sizeof(double));
}

template <int NW, typename At>
static int apply_w_launch(const FactorBatch &batch, const At &at, const dim3 &grid, int max_nb, int round, hipStream_t st) {
    const size_t bytes = (size_t)max_nb * 16 * 64 * sizeof(float);
    static size_t granted = 0;
    int rc = grant_dynamic_lds(reinterpret_cast<const void *>(apply_w_kernel<NW, At>), bytes, &granted, "apply_w attribute");
    if (rc != DLCX_OK) return rc;
    Timed timed(KID_APPLY_W, st);
    hipLaunchKernelGGL((apply_w_kernel<NW, At>), grid, dim3(64 * NW), bytes, st, batch, at, round);
    return check_launch("apply_w");
}

static int cholqr_round(const FactorBatch &batch, int round, hipStream_t st) {
    FactorBatch summed;  // the same factors with their Gram sums in one chunk
    int rc = launch_gram_partials_batch(batch, &summed, round, st);
    if (rc != DLCX_OK) return rc;
    int max_nb = 1;
    for (int i = 0; i < batch.n; ++i) {
        const int nb = (batch.it[i].r + 15) / 16;
        if (nb > max_nb) max_nb = nb;
    }
    {
        // A wavefront for the diagonal blocks, up to seven for the others; blocks of each: 1 up to r = 64, 2 up to
        // r = 80, 6 up to r = 144, else 18.  (Slots without a block load and add like the others: at r = 48 two to
        // a wavefront took 31.0 us, one 29.5.)
        Timed timed(KID_CHOL, st);
        const int others = max_nb * (max_nb - 1) / 2, dealt = kCT / 64 - 1;
        const dim3 grid((unsigned)batch.n), threads((unsigned)(1 + (others < dealt ? others : dealt)) * 64);
        static_assert(kMaxBlocks <= 2 * (kCT / 64), "two blocks on the diagonal for every wavefront at most");
        static_assert(6 * 7 >= (kSumRank / 16) * (kSumRank / 16 - 1) / 2, "ranks that sum chunks have at most 6");
        static_assert(18 / 3 * 20 >= kMaxBlocks * (kMaxBlocks - 1) / 2, "blocks of the largest rank");
        if (others <= dealt)
            hipLaunchKernelGGL(chol_inverse_kernel<1>, grid, threads, 0, st, summed, round);
        else if (others <= 2 * dealt)
            hipLaunchKernelGGL(chol_inverse_kernel<2>, grid, threads, 0, st, summed, round);
        else if (others <= 6 * dealt)
            hipLaunchKernelGGL(chol_inverse_kernel<6>, grid, threads, 0, st, summed, round);
        else
            hipLaunchKernelGGL(chol_inverse_kernel<18>, grid, threads, 0, st, summed, round);
        rc = check_launch("chol_inverse");
    }
    if (rc != DLCX_OK) return rc;
    auto rows = [](const FactorItem &it) { return ceil_div(it.L, 64); };
    return for_places(batch, kMostRows, 1, rows, [&](auto at, int x, int y) {
        using At = decltype(at);
        const dim3 grid((unsigned)x, (unsigned)y);
        return max_nb > 8 ? apply_w_launch<8, At>(batch, at, grid, max_nb, round, st)
                          : apply_w_launch<4, At>(batch, at, grid, max_nb, round, st);
    });
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
    size_t bytes = 0;
    bool small = true;
    for (int i = 0; i < batch.n; ++i) {
        const FactorItem &it = batch.it[i];
        small = small && it.r <= kSmallOrthRank && it.L <= kSmallOrthLength && small_bytes(it.L, it.r) <= kSmallFloats * sizeof(float);
        if (small && small_bytes(it.L, it.r) > bytes) bytes = small_bytes(it.L, it.r);
    }
    if (small) {
        static size_t granted = 0;
        int rc = grant_dynamic_lds(reinterpret_cast<const void *>(orth_small_kernel), bytes, &granted, "orth_small attribute");
        if (rc != DLCX_OK) return rc;
        Timed timed(KID_CHOL, st);
        hipLaunchKernelGGL(orth_small_kernel, dim3((unsigned)batch.n), dim3(kSmallThreads), bytes, st, batch);
        return check_launch("orth_small");
    }
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
