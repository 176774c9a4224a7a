// r' of Alg. 3 for one matrix: the smallest k whose k largest eigenvalues of S = Q_bar^T Q_bar
// hold at least tau of the trace (with P_hat orthonormal these are the squared singular values of
// the decompressed average).  S is accumulated in fp64 (same partial-sum kernel as the
// orthonormalisation).  Everything after it is fp64 too:
//   tridiag_kernel       Householder reduction to tridiagonal form, one workgroup per matrix
//   eigenvalues          every eigenvalue by multisection on the Sturm sequence: G lanes evaluate
//                        G points of an interval at once, so a round narrows it G + 1 times; only
//                        as far as it takes to tell which sums hold the share
//   count                prefix sum over the eigenvalues (they come out in order) and count
// Up to rank 64 the last two follow in the same workgroup; above, eigenvalue_bounds_kernel and, where those leave
// it open, eigenvalues_kernel spread them over the GPU (one wavefront per eigenvalue) and count_kernel finishes.
#include <type_traits>

#include "common.h"

namespace dlcx {

constexpr int kTT = 256;             // threads of the reduction up to kFusedRank
constexpr int kTri = 512;            // and above
constexpr int kFusedRank = 64;       // ranks up to here finish in the same workgroup
constexpr int kTail = 64;            // rows that one wavefront reduces at most

// the fp64 value of the lane that DPP control `kCtrl` pairs this lane with (inside rows of 16)
template <int kCtrl>
__device__ __forceinline__ double dpp(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, kCtrl, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), kCtrl, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor7 = 0x141, kXor15 = 0x140;
constexpr int kRowShl1 = 0x101;  // from the lane after it, the last of a row of 16: zero

__device__ __forceinline__ double from_halves(uint32_t lo, uint32_t hi) {
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// sum of a over both halves of the wavefront in lanes 0 - 31, of b in lanes 32 - 63
__device__ __forceinline__ double add_halves(double a, double b) {
    const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
    return from_halves(lo[0], hi[0]) + from_halves(lo[1], hi[1]);
}
// sum of a over a pair of rows of 16 lanes in the even row, of b in the odd row
__device__ __forceinline__ double add_rows(double a, double b) {
    const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
    return from_halves(lo[0], hi[0]) + from_halves(lo[1], hi[1]);
}
// sum over the wavefront, in every lane
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp<kXor1>(x);
    x += dpp<kXor2>(x);
    x += dpp<kXor7>(x);
    x += dpp<kXor15>(x);
    x = add_rows(x, x);
    return add_halves(x, x);
}

// Four sums over the 16 lanes of a row at once: the lanes halve the values among themselves as they add, lane t
// ends up with the sum of value t / 4.
template <int kCtrl, int M>
__device__ __forceinline__ void halve(double (&v)[4], bool up) {
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const double keep = up ? v[i + M] : v[i], send = up ? v[i] : v[i + M];
        v[i] = keep + dpp<kCtrl>(send);
    }
}
__device__ __forceinline__ double row_sums(double (&v)[4], int t) {
    halve<kXor15, 2>(v, t & 8);
    halve<kXor7, 1>(v, t & 4);
    v[0] += dpp<kXor2>(v[0]);
    v[0] += dpp<kXor1>(v[0]);
    return v[0];
}

// The tridiagonal matrix as the Sturm sequence reads it: t[i] = (d_i, -e_i^2), e_i between i - 1
// and i, scaled to magnitudes of at most one.
__device__ __forceinline__ double2 sturm_term(double d, double e) {
    // an off-diagonal below 2^-60 of the scale counts as that: p_i = 0 with e = 0 would end the
    // sequence, and 2^-60 moves no eigenvalue by more than the arithmetic does
    return make_double2(d, -fmax(e * e, 0x1p-120));
}

// The table is filled up to whole blocks of 16 terms, and one half block more is read, never used:
// diagonal elements above every x, coupled to nothing, which add no sign change.
constexpr int kSturmPad = 24;
__device__ __forceinline__ int sturm_blocks(int r) { return (r + 15) >> 4; }
__device__ __forceinline__ double2 sturm_fill() { return make_double2(4.0, 0.0); }

// Number of eigenvalues below x: sign changes of p_i = (d_i - x) p_{i-1} - e_i^2 p_{i-2}, where the
// quotients p_i / p_{i-1} would need a division per term.  The sign bits are collected and compared
// 16 at a time; every eight terms the pair is scaled back by the larger of the two (one may be exactly
// zero: x on the diagonal of decoupled rows).  A term is at most 5 x the larger of the two before it, and
// the step from pair to pair has the determinant e^2 >= 2^-120: over eight the larger one grows at most
// 2^19 x and shrinks to no less than 2^-979, so nothing overflows or vanishes between.  Eight terms are
// read while the eight before are worked on.
__device__ __forceinline__ int count_below(const double2 *t, int blocks, double x) {
    double p0 = 0.0, p1 = 1.0;  // t[0].y multiplies p0
    uint32_t signs = 0;
    int cnt = 0;
    double2 even[8], odd[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) even[u] = t[u];
    auto eight = [&](const double2 (&c)[8]) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double p = fma(c[u].x - x, p1, c[u].y * p0);
            signs = __builtin_amdgcn_alignbit(signs, (uint32_t)((uint64_t)__double_as_longlong(p) >> 32), 31);
            p0 = p1;
            p1 = p;
        }
        const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
        p0 = ldexp(p0, ex);
        p1 = ldexp(p1, ex);
    };
    for (int i = 0; i < blocks; ++i) {
#pragma unroll
        for (int u = 0; u < 8; ++u) odd[u] = t[16 * i + 8 + u];
        __builtin_amdgcn_sched_barrier(0);
        eight(even);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) even[u] = t[16 * i + 16 + u];
        __builtin_amdgcn_sched_barrier(0);
        eight(odd);
        cnt += __popc((signs ^ (signs >> 1)) & 0xffffu);  // the 16 newest against those before them
    }
    return cnt;
}

// Bounds lo, hi of the c-th largest eigenvalue (c from 0), inside [-1, 1], narrowed `rounds` times by groups of G
// lanes, every lane of the wavefront calling: G points of the interval at once, so a round narrows it G + 1 times.
template <int G>
__device__ __forceinline__ void narrow(const double2 *t, int r, int c, double &lo, double &hi, int lane, int rounds) {
    const int below = r - 1 - c;  // eigenvalues smaller than the one wanted
    const int sub = lane & (G - 1), base = lane - sub;
    constexpr uint64_t mask = G == 64 ? ~0ull : (1ull << (G & 63)) - 1;
    for (int itn = 0; itn < rounds; ++itn) {
        const double step = (hi - lo) * (1.0 / (double)(G + 1));
        const double x = fma((double)(sub + 1), step, lo);
        const bool above = count_below(t, sturm_blocks(r), x) > below;  // x is above the eigenvalue
        const uint64_t m = (__ballot(above) >> base) & mask;
        const int first = m ? __builtin_ctzll(m) : G;  // points 0 .. first - 1 are not
        const double nlo = first > 0 ? fma((double)first, step, lo) : lo;
        const double nhi = first < G ? fma((double)(first + 1), step, lo) : hi;
        lo = nlo;
        hi = nhi;
    }
}
// Rounds to an interval of less than 2^-56, 2 (G + 1)^-n: the sums that decide r' are at least 1/2 and rounded at
// 2^-54, so an eigenvalue that is zero, or vanishes beside the others, then adds nothing to them.  After the first
// kEarly of them, at 2^-19 .. 2^-23, the bounds nearly always tell already which sums hold the share (decided()).
template <int G>
struct Rounds {
    static constexpr int kAll = G == 64 ? 10 : G == 32 ? 12 : G == 16 ? 14 : G == 8 ? 18 : 25;
    static constexpr int kEarly = G == 64 ? 4 : G == 32 ? 4 : G == 16 ? 5 : G == 8 ? 7 : 9;
};
__device__ __forceinline__ double eigenvalue(double lo, double hi) { return fmax(0.5 * (lo + hi), 0.0); }

// r' from bounds of the r eigenvalues in descending order, N a lane: value 64 q + lane is between lo[q] and hi[q].
// Returns -1 where the bounds leave open whether one of the sums holds tau of the total: what count_share
// makes of values inside the bounds it then returns, whatever they are.  The k largest hold the share if
// (1 - tau) of their sum is at least tau of the sum of the others; 2^-40 of the total is beyond all roundings.
template <int N>
__device__ __forceinline__ int decided(const double (&lo)[N], const double (&hi)[N], int r, double tau, int lane) {
    double ls[N], hs[N], lt = 0.0, ht = 0.0;  // the sums up to a value, the totals
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const bool on = 64 * q + lane < r;
        ls[q] = on ? fmax(lo[q], 0.0) : 0.0;
        hs[q] = on ? fmax(hi[q], 0.0) : 0.0;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double l = __shfl_up(ls[q], off, 64), h = __shfl_up(hs[q], off, 64);
            ls[q] += lane >= off ? l : 0.0;
            hs[q] += lane >= off ? h : 0.0;
        }
        ls[q] += lt;
        hs[q] += ht;
        lt = read_lane(ls[q], 63);
        ht = read_lane(hs[q], 63);
    }
    const double slack = 0x1p-40 * ht;
    int k = 0;
    bool open = false;
#pragma unroll
    for (int q = N - 1; q >= 0; --q) {
        const bool on = 64 * q + lane < r;
        const bool yes = (1.0 - tau) * ls[q] >= tau * (ht - hs[q]) + slack;
        const bool no = (1.0 - tau) * hs[q] + slack < tau * (lt - ls[q]);
        open = open || __ballot(on && !yes && !no) != 0;
        const uint64_t m = __ballot(on && yes);
        if (m) k = 64 * q + __builtin_ctzll(m) + 1;
    }
    return open || k == 0 ? -1 : k;
}

// smallest k whose k largest of the descending values (in LDS, zeros behind them up to a multiple of 64)
// hold at least tau of their sum (0: all zero), by one wavefront.  Every lane adds them all up one after the other, largest first, and keeps the
// partial sums that fall to it: for tau = 1 it matters that the total is the last of those sums.
__device__ __forceinline__ int32_t count_share(const double *eig, int r, double tau, int lane) {
    double keep[DLCX_MAX_RANK / 64] = {0.0, 0.0, 0.0, 0.0}, cum = 0.0;
#pragma unroll
    for (int q = 0; q < DLCX_MAX_RANK / 64; ++q) {
        for (int c = 0; c < 64 && 64 * q + c < r; c += 16) {  // sixteen read at a time
            double e[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) e[u] = eig[64 * q + c + u];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                cum += e[u];
                keep[q] = lane == c + u ? cum : keep[q];
            }
        }
    }
    int32_t k = r;
#pragma unroll
    for (int q = DLCX_MAX_RANK / 64 - 1; q >= 0; --q) {
        const uint64_t m = __ballot(keep[q] >= tau * cum && 64 * q + lane < r);
        if (m) k = 64 * q + __builtin_ctzll(m) + 1;
    }
    return cum > 0.0 ? k : 0;
}

// The Householder reflection of a row whose first element right of the diagonal is x0 and whose
// others have `tail` as their sum of squares.  With s = x0^2 + tail: alpha = -+sqrt(s), v = row with
// v_0 = x0 - alpha, beta = 2 / |v|^2 = 1 / (s + |x0| sqrt(s)); v_rsq_f64 and v_rcp_f64 with two
// Newton steps each are full fp64.  beta = 0: nothing to reflect, alpha = x0.  (Below 2^-960 a tail is
// rounding of roundings: S comes from fp32 values, its entries are above 2^-300 or zero; and
// v_rsq_f64 needs a normal number.)
struct Reflection {
    double alpha, beta;
};
__device__ __forceinline__ Reflection reflection(double x0, double tail) {
    const double s = fma(x0, x0, tail);
    double y = __builtin_amdgcn_rsq(s);
    y = fma(0.5 * y, fma(-s * y, y, 1.0), y);
    y = fma(0.5 * y, fma(-s * y, y, 1.0), y);
    const double norm = s * y, den = fma(fabs(x0), norm, s);
    double beta = __builtin_amdgcn_rcp(den);
    beta = fma(fma(-den, beta, 1.0), beta, beta);
    beta = fma(fma(-den, beta, 1.0), beta, beta);
    const bool reflect = tail > 0x1p-960;
    return Reflection{reflect ? -copysign(norm, x0) : x0, reflect ? beta : 0.0};
}

// Gershgorin interval of the tridiagonal matrix (tri[i] = d_i, e_{i-1}), by one wavefront, scaled by
// 2^ex, the power of two that puts every magnitude at one or below.
struct Interval {
    double lo, hi;
    int ex;
};
__device__ __forceinline__ Interval gershgorin(const double2 *tri, int r, int lane) {
    double lo = tri[0].x, hi = lo;
    for (int i = lane; i < r; i += 64) {
        const double rad = (i > 0 ? fabs(tri[i].y) : 0.0) + (i + 1 < r ? fabs(tri[i + 1].y) : 0.0);
        lo = fmin(lo, tri[i].x - rad);
        hi = fmax(hi, tri[i].x + rad);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off, 64));
        hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    const double big = fmax(fabs(lo), fabs(hi));
    const int ex = big > 0.0 && big < 1e300 ? -__builtin_amdgcn_frexp_exp(big) : 0;
    return Interval{ldexp(lo, ex), ldexp(hi, ex), ex};
}

// What tridiag_kernel leaves in FactorItem::g above rank 64: the Sturm table with all that count_below reads,
// from double 0; then lo, hi and the number of rows that are not zero.  Behind them the other kernels' part, written
// while the table is read: whether r' is open, bounds of every eigenvalue, the eigenvalues (still scaled: r' does
// not depend on a power of two).
constexpr int kTableTerms = DLCX_MAX_RANK + 8;
static_assert(kTableTerms >= (DLCX_MAX_RANK + 15) / 16 * 16 + 8, "whole blocks and the half block after them");
static_assert(2 * kTableTerms + 8 + 3 * DLCX_MAX_RANK <= (kFusedRank + 2) * (kFusedRank + 2), "room in the smallest g");
__device__ __forceinline__ double2 *tri_of(const FactorItem &it) { return reinterpret_cast<double2 *>(it.g); }
__device__ __forceinline__ double *bounds_of(const FactorItem &it) { return it.g + 2 * kTableTerms; }
__device__ __forceinline__ int live_of(const FactorItem &it) { return __builtin_amdgcn_readfirstlane((int)bounds_of(it)[2]); }
__device__ __forceinline__ double *open_of(const FactorItem &it) { return it.g + 2 * kTableTerms + 7; }
__device__ __forceinline__ double *eig_of(const FactorItem &it) { return it.g + 2 * kTableTerms + 8; }
__device__ __forceinline__ double *low_of(const FactorItem &it) { return eig_of(it) + DLCX_MAX_RANK; }
__device__ __forceinline__ double *high_of(const FactorItem &it) { return eig_of(it) + 2 * DLCX_MAX_RANK; }

// The Gram sums over chunk c of a factor of at most 16 columns by the workgroup that goes on with them,
// a quarter of the chunk per wavefront, as gram_partial_kernel forms them, bit for bit (whether a factor's
// sums come from there depends on the batch).  Up to kSmallGramLength rows that is no longer than a launch before
// this one, us without | with it, from the host: 512 x 8 9.7 | 11.7, 512 x 16 13.2 | 15.3, 1024 x 8 11.8 | 11.9, 1024 x
// 16 15.4 | 15.7; in a graph 512 x 8 10.3 | 11.9, 1024 x 8 12.4 | 12.1, 1024 x 16 16.1 | 15.7.  Above it is longer, as a
// chunk takes 2 us (in a graph): 1040 x 8 13.1 | 12.2, 1536 x 8 14.6 | 12.4, 1536 x 16 18.2 | 15.7, 2048 x 16 20.4 | 16.1.
constexpr int kSmallGramRank = 16;
constexpr int kSmallGramLength = 1024;
__device__ __forceinline__ void small_gram(const FactorItem &it, int c, double (&gram)[4][kSmallGramRank][kSmallGramRank + 1]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g = lane >> 4, L = (int)it.L, begin = (4 * c + wave) * kGramQuarter;
    const float *row = it.f + (int64_t)(col < it.r ? col : it.r - 1) * L + 4 * g;
    float4 x[kGramQuarter / 16];
#pragma unroll
    for (int u = 0; u < kGramQuarter / 16; ++u)
        x[u] = *reinterpret_cast<const float4 *>(row + (begin + 16 * u < L ? begin + 16 * u : 0));
    f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < kGramQuarter / 16; ++u) {
        if (begin + 16 * u >= L) break;
        acc = gram_step(x[u], acc);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) gram[wave][4 * v + g][col] = acc[v];
}

// ---------------------------------------------------------------------------------------------
// Householder reduction by one wavefront, rows in lanes, columns in registers, no barrier and no LDS but for the
// result.  A step, with x the column that is reflected (v: x below the diagonal, its first element moved by c):
//   u = S x_tail and the sums over |x_tail|^2 and x_tail . u do not wait for the reflection, they run beside it:
//   S v = u + c S_1 and v . S v = x_tail . u + c (2 u_1 + c S_11), with S_1 the next column and u_1 = S_1 . x_tail;
//   S -= v w^T + w v^T, the next column first.
// An element of x, v, w along the columns comes from one lane of each row of 16 as the operand of the product
// (row_newbcast); the rows are dealt to the lanes so that such a register is a copy of rows of lanes of the
// vector itself.  After four steps rows and columns are renumbered: register and lane indices are constants.
// ---------------------------------------------------------------------------------------------
// What other lanes read (DPP, permlane, readlane) has to be up to two wait states behind the vector instruction that
// wrote it.  The compiler sees to that between its own instructions but does not look into these: two at the front
// for src, w and v, and what is read so of their results goes through settle() before.  (Two behind every one of them:
// 2048 x 64 64.7 | 68.4 us.)  Results are written before the last operand is read: no register in common.
__device__ __forceinline__ void settle(double &x) { asm("s_nop 1" : "+v"(x)); }
__device__ __forceinline__ void settle8(double *t) {
    asm("s_nop 1" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]), "+v"(t[7]));
}
// acc[i % 2] += element C + i of src (one lane of each row of 16) * by[i], i = 0 .. 3.  Not for other lanes to read.
template <int C>
__device__ __forceinline__ void dot_bcast4(double (&acc)[2], double src, const double *by) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %2, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc[0]), "+&v"(acc[1])
        : "v"(src), "v"(by[0]), "v"(by[1]), "v"(by[2]), "v"(by[3]), "n"(C), "n"(C + 1), "n"(C + 2), "n"(C + 3));
}
// t[i] += (element C + i of w) * a + (element C + i of v) * b, i = 0 .. 3
template <int C>
__device__ __forceinline__ void update_bcast4(double *t, double w, double a, double v, double b) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %4, %5 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %4, %5 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %6, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %6, %7 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %6, %7 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %6, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf"
        : "+&v"(t[0]), "+&v"(t[1]), "+&v"(t[2]), "+&v"(t[3])
        : "v"(w), "v"(a), "v"(v), "v"(b), "n"(C), "n"(C + 1), "n"(C + 2), "n"(C + 3));
}
struct Two {
    double a, b;
};
// .a: the lower half of the wavefront in both halves, .b: the upper
__device__ __forceinline__ Two halves_of(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return Two{from_halves(lo[0], hi[0]), from_halves(lo[1], hi[1])};
}
// .a: the even row of each pair of rows of 16 lanes in both, .b: the odd one
__device__ __forceinline__ Two rows_of(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return Two{from_halves(lo[0], hi[0]), from_halves(lo[1], hi[1])};
}

// Up to 32 rows: row 2 m + b in lanes 16 b + m and 32 + 16 b + m, the lower half of the wavefront with the even
// columns, the upper with the odd ones: t[c] is column 2 c + h.
struct Rows32 {
    static __device__ __forceinline__ int row(int lane) { return 2 * (lane & 15) + ((lane >> 4) & 1); }
    static constexpr int lane(int row) { return (row >> 1) + 16 * (row & 1); }
    static __device__ __forceinline__ double sum(double x) {
        x += dpp<kXor1>(x);
        x += dpp<kXor2>(x);
        x += dpp<kXor7>(x);
        x += dpp<kXor15>(x);
        return add_rows(x, x);
    }
    static __device__ __forceinline__ double gather(double x) { return add_halves(x, x); }
    template <int J>
    static __device__ __forceinline__ double column(double *t) {
        settle(t[J >> 1]);
        const Two x = halves_of(t[J >> 1]);
        return (J & 1) ? x.b : x.a;
    }
    static __device__ __forceinline__ void spread(double x, int lane, double (&to)[1]) {
        const Two r = rows_of(x);
        to[0] = lane < 32 ? r.a : r.b;
    }
    // the lane that holds element `row` of a spread vector
    static __device__ __forceinline__ bool holds(int lane, int q, int row) { return (lane >> 5) == (row & 1) && (lane & 15) == (row >> 1); }
    static constexpr int kSpread = 1;
    static constexpr int kSteps = 2;  // to a register of columns
};
// Up to 64 rows: row 4 m + b in lane 16 b + m, t[16 q + c] is column 4 c + q.
struct Rows64 {
    static __device__ __forceinline__ int row(int lane) { return 4 * (lane & 15) + (lane >> 4); }
    static constexpr int lane(int row) { return (row >> 2) + 16 * (row & 3); }
    static __device__ __forceinline__ double sum(double x) { return wave_sum(x); }
    static __device__ __forceinline__ double gather(double x) { return x; }
    template <int J>
    static __device__ __forceinline__ double column(double *t) {
        settle(t[16 * (J & 3) + (J >> 2)]);
        return t[16 * (J & 3) + (J >> 2)];
    }
    static __device__ __forceinline__ void spread(double x, int, double (&to)[4]) {
        const Two r = rows_of(x), even = halves_of(r.a), odd = halves_of(r.b);
        to[0] = even.a;
        to[1] = odd.a;
        to[2] = even.b;
        to[3] = odd.b;
    }
    static __device__ __forceinline__ bool holds(int lane, int q, int row) { return q == (row & 3) && (lane & 15) == (row >> 2); }
    static constexpr int kSpread = 4;
    static constexpr int kSteps = 4;
};

// Steps k, k + 1, .. up to `stop`, a multiple of Rows::kSteps away, or until row r - 1 is reached; C registers of
// each spread vector's columns are in use (the others are done).  x: the column of step k.  tri: the result's place
// for lane 0, places of no use for the others.
template <typename Rows, int C>
__device__ __forceinline__ void reduce_steps(double *t, double &x, int &k, int stop, int r, double2 *tri, int lane) {
    constexpr int Q = Rows::kSpread;
    const int row = Rows::row(lane);
    for (; k < stop && k < r; k += Rows::kSteps) {
        unrolled<Rows::kSteps>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            const double dk = read_lane(x, Rows::lane(s));
            tri[k + s].x = dk;
            if (k + s + 1 >= r) return;
            const double x0 = read_lane(x, Rows::lane(s + 1)), xt = row > s + 1 ? x : 0.0;
            double xb[Q];
            Rows::spread(xt, lane, xb);
            double acc[2] = {0.0, 0.0};
            unrolled<Q>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                unrolled<C / 4>([&](auto cc) { dot_bcast4<4 * decltype(cc)::value>(acc, xb[q], t + 16 * q + 4 * decltype(cc)::value); });
            });
            const double tail = Rows::sum(xt * xt);
            const double u = Rows::gather(acc[0] + acc[1]);
            const double s1 = Rows::template column<s + 1>(t);
            const double xu = Rows::sum(xt * u);
            const Reflection f = reflection(x0, tail);
            const double c = x0 - f.alpha;
            tri[k + s + 1].y = f.alpha;
            const double vp = fma(c, fma(c, read_lane(s1, Rows::lane(s + 1)), 2.0 * read_lane(u, Rows::lane(s + 1))), xu);
            const double kk = 0.5 * f.beta * (f.beta * vp);  // (beta^2 may overflow)
            const double v = row == s + 1 ? c : xt, p = fma(c, s1, u);
            const double w = row > s ? fma(f.beta, p, -kk * v) : 0.0;
            double wb[Q];
            Rows::spread(w, lane, wb);
#pragma unroll
            for (int q = 0; q < Q; ++q) xb[q] = Rows::holds(lane, q, s + 1) ? c : xb[q];  // v
            unrolled<Q>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                unrolled<C / 4>([&](auto cc) {
                    update_bcast4<4 * decltype(cc)::value>(t + 16 * q + 4 * decltype(cc)::value, wb[q], -v, xb[q], -w);
                });
            });
            x = fma(c, -w, fma(read_lane(w, Rows::lane(s + 1)), -v, s1));  // as the same element of t
        });
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int c = 0; c < C; c += 8) settle8(t + 16 * q + c);
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int c = 0; c < C; ++c) t[16 * q + c] = c + 1 < C ? dpp<kRowShl1>(t[16 * q + c + 1]) : 0.0;
        x = dpp<kRowShl1>(x);
    }
}
// The reduction of the r x r matrix element(i, j), r <= 32: d_i and the off-diagonal before it to tri[i]
template <typename F>
__device__ __forceinline__ void reduce32(F &&element, int r, double2 *tri, int lane) {
    double t[16];
    const int row = Rows32::row(lane), h = lane >> 5;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const int j = 2 * c + h;
        const double e = element(row < r ? row : 0, j < r ? j : 0);
        t[c] = row < r && j < r ? e : 0.0;
    }
    double x = Rows32::column<0>(t);
    int k = 0;
    if (r > 16) reduce_steps<Rows32, 16>(t, x, k, (r - 15) & ~1, r, tri, lane);  // to 16 rows or fewer
    reduce_steps<Rows32, 8>(t, x, k, r, r, tri, lane);
}

// The same for r <= 64; the last 32 rows go through `sm`, which element() may read as well
template <typename F, int P>
__device__ __forceinline__ void reduce64(F &&element, int r, double2 *tri, double (*sm)[P], int lane) {
    if (r <= 32) {
        reduce32(element, r, tri, lane);
        return;
    }
    double t[64];
    const int row = Rows64::row(lane);
#pragma unroll
    for (int j = 0; j < 64; ++j) {
        const double e = element(row < r ? row : 0, j < r ? j : 0);
        t[16 * (j & 3) + (j >> 2)] = row < r && j < r ? e : 0.0;
    }
    double x = t[0];
    int k = 0;
    reduce_steps<Rows64, 16>(t, x, k, (r - 29) & ~3, r, tri, lane);  // to 32 rows or fewer
#pragma unroll
    for (int j = 0; j < 32; ++j)
        if (row < 32) sm[row][j] = t[16 * (j & 3) + (j >> 2)];
    wave_sync();
    reduce32([&](int i, int j) { return sm[i][j]; }, r - k, tri + k, lane);
}

// Householder reduction of S to tridiagonal form, one workgroup per matrix, S in registers.
// S is cut into 16 x 16 tiles, of which the upper ones (x <= y) exist; thread (h, ti, tj) holds element
// (ti, tj) of the tiles whose column y has parity h.  An off-diagonal tile serves S v twice, along its
// rows and its columns.  Step k, with v of row k in LDS:
//   S v      row parts added over the 16 lanes of tj, column parts over ti: four rows of lanes in a
//            wavefront, four wavefronts and two parities in LDS                              | barrier
//   p = S v  the parts added up, two lanes per entry                                         | barrier
//   S -= v w^T + w v^T  with w = beta p - (beta^2 v.p / 2) v, formed where it is used; before its own
//            share one wavefront works out the next v and beta from row k + 1, which the update before
//            has left in LDS                                                                 | barrier
// Rows that are done have zeros in v and w; groups of four tile rows that are done are skipped (a branch for
// every row took as long as the work it saved).
// The last kTail rows go to one wavefront (reduce64), 0.45 - 0.7 us a step and no barrier, where they took 1.2 - 2
// here: whole calls, us before | after (the 20 - 30 of the eigenvalue bounds in it), 2048 x 66 133 | 76, 8192 x 100
// 196 | 149, 5008 x 130 302 | 226, seven factors at r = 190 471 | 407, at 256 739 | 672.
// Bound by the instructions of a step, two wavefronts to a SIMD, and by the chain of the reflection, 191
// steps in a row at r = 256.  Eight wavefronts of 256 registers, 144 of them tiles at r = 256: with one wavefront per
// SIMD half of the tiles sat in the accumulator file, which vector instructions cannot name, two moves for
// every use.  v and w along the rows come from one lane of each row of 16 (row_bcast): read from LDS row by
// row they kept the LDS busy for a third of a step.  Seven factors at r = 256: 2.4 us a step, of which
// S v 0.75, sums and barriers 0.45, the reflection 0.5 and the update behind it 0.4 (one wavefront per SIMD:
// 783 us; whole tile rows dealt to the wavefronts, which need fewer sums across lanes but differ in work and
// branch at every tile: 725 us).
template <int NT>
__global__ __launch_bounds__(kTri, 1) void tridiag_kernel(FactorBatch batch) {
    constexpr int R = 16 * NT;
    constexpr int N = NT / 2;   // tile columns of one parity
    constexpr int Q = R / 64;   // entries per lane where one wavefront has a whole row
    constexpr int W = kTri / 64;
    __shared__ double vbuf[2][R + 1];   // v of even and odd steps, zeros up to the diagonal
    __shared__ double betas[2];         // 0: the row is tridiagonal already
    __shared__ double arow[2][R + 1];   // row k + 1 of S before the update of step k, from the diagonal on
    __shared__ double pbuf[R + 1];
    __shared__ double rowpart[2][R];
    __shared__ double colpart[4][R];
    __shared__ double2 tri[R + kSturmPad], unused[64 + kTail + kSturmPad];  // d_k and the off-diagonal element before it
    __shared__ double sm[kTail][kTail + 1];  // the last rows
    __shared__ int order[R];            // the rows of S that are not zero
    __shared__ int counts[W];
    const FactorItem it = batch.it[blockIdx.x];
    const int nchunks = it.nchunks;
    const double *__restrict__ part = it.part;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int par = wave & 1, quarter = wave >> 1;  // parity h; ti / 4
    const int tj = lane & 15, g = lane >> 4, ti = quarter * 4 + g;
    const int row_lane = tj < NT ? tj : 0;
    const int64_t pitch = it.r, rr = pitch * pitch;
    if (it.r <= kFusedRank) return;

    // The zero columns of the factor: left out, their eigenvalues are zero.  (Reflected with the others
    // they would come back as rounding, and count at tau = 1.)
    bool on = false, odd = false;
    if (tid < it.r) {
        double s = 0.0;
        for (int c = 0; c < nchunks; ++c) s += part[tid * pitch + tid + c * rr];
        on = s != 0.0;
        odd = !(s < __builtin_inf());
    }
    const uint64_t mask = __ballot(on);
    const bool wave_odd = __ballot(odd) != 0;  // a NaN or an infinity in the factor: no rows, r' = 0
    if (lane == 0) counts[wave] = wave_odd ? -kTri : __popcll(mask);
    if (tid < 2) {
        vbuf[tid][R] = 0.0;
        arow[tid][R] = 0.0;
        pbuf[R] = 0.0;
    }
    __syncthreads();
    int before = 0, r = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        before += q < wave ? counts[q] : 0;
        r += counts[q];
    }
    if (on && before >= 0) order[before + __popcll(mask & ((1ull << lane) - 1))] = tid;
    r = __builtin_amdgcn_readfirstlane(r < 0 ? 0 : r);
    __syncthreads();

    // t[x][i]: tile (x, 2 i + h).  Where x is odd, i starts with the diagonal tile of h = 1; beside it
    // h = 0 has the tile left of the diagonal, which takes no part in S v.
    double t[NT][N];
#pragma unroll
    for (int x = 0; x < NT; ++x) {
        const int a = 16 * x + ti, oa = a < r ? order[a] : 0;
#pragma unroll
        for (int i = x / 2; i < N; ++i) {
            const int b = 16 * (2 * i + par) + tj, ob = b < r ? order[b] : 0;
            const bool in = a < r && b < r;  // order[] rises
            const double *src = part + (in ? (oa < ob ? oa * pitch + ob : ob * pitch + oa) : 0);
            double s = src[0];
            for (int c = 1; c < nchunks; ++c) s += src[c * rr];
            t[x][i] = in ? s : 0.0;
        }
    }
    // Row `row`, whose tile row is x, from its tile on.
    auto keep_row = [&](auto xc, int row) {
        constexpr int x = decltype(xc)::value;
        if (((row & 15) >> 2) != quarter || g != (row & 3)) return;
        double *dst = &arow[row & 1][tj];
#pragma unroll
        for (int i = x / 2; i < N; ++i)
            if (i > x / 2 || x % 2 == 0 || par == 1) dst[16 * (2 * i + par)] = t[x][i];
    };
    // The reflection of row c, by one wavefront, R / 64 entries per lane (lv, lw: v and w there; vc, v1, wc,
    // w1: at c and c + 1; all zero for the first).  c + 1 may be R: nothing is right of the last row.
    auto reflect = [&](int c, const double (&lv)[Q], const double (&lw)[Q], double vc,
                       double wc, double v1, double w1) {
        const double *ar = arow[c & 1];
        double a[Q], tail = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const double x = fma(-lv[q], wc, fma(-lw[q], vc, ar[lane + 64 * q]));
            a[q] = lane + 64 * q > c + 1 ? x : 0.0;  // arow has nothing left of the diagonal tile
            tail = fma(a[q], a[q], tail);
        }
        const double x0 = fma(-v1, wc, fma(-w1, vc, ar[c + 1])), d = fma(-vc, wc, fma(-wc, vc, ar[c]));
        const Reflection f = reflection(x0, wave_sum(tail));
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int e = lane + 64 * q;
            const double y = e == c + 1 ? x0 - f.alpha : a[q];
            vbuf[c & 1][e] = f.beta == 0.0 ? 0.0 : y;
        }
        if (lane == 0) {
            betas[c & 1] = f.beta;
            tri[c].x = d;
            if (c + 1 < R) tri[c + 1].y = f.alpha;
        }
    };
    keep_row(std::integral_constant<int, 0>(), 0);
    keep_row(std::integral_constant<int, 0>(), 1);
    __syncthreads();
    const int stop = r > kTail ? r - kTail : 0;
    if (wave == 0 && stop > 0) {
        const double zero[Q] = {};
        reflect(0, zero, zero, 0.0, 0.0, 0.0, 0.0);
    }
    __syncthreads();
    for (int k = 0; k < stop; ++k) {
        const double *v = vbuf[k & 1];
        // v along the columns of this thread's tiles and, from lane x of its row, along their rows
        double cv[N];
#pragma unroll
        for (int i = 0; i < N; ++i) cv[i] = v[16 * (2 * i + par) + tj];
        const double rv = v[16 * row_lane + ti];
        {
            const int live = (k + 1) >> 4;  // tile rows and columns before it are done
            double cp[(N + 3) / 4 * 4] = {};
            unrolled<NT / 4>([&](auto bc) {
                constexpr int x0 = 4 * decltype(bc)::value;
                if (x0 + 3 < live) return;
                double rp[4];
                unrolled<4>([&](auto uc) {
                    constexpr int u = decltype(uc)::value, x = x0 + u, i0 = x / 2;
                    const double rx = row_bcast<x>(rv);
                    // the first tile: on the diagonal (row part only) for h = x % 2; none for x odd and h = 0
                    rp[u] = t[x][i0] * (x % 2 == 0 || par == 1 ? cv[i0] : 0.0);
                    if (x % 2 == 0) cp[i0] = fma(t[x][i0], par == 1 ? rx : 0.0, cp[i0]);
#pragma unroll
                    for (int i = i0 + 1; i < N; ++i) {
                        rp[u] = fma(t[x][i], cv[i], rp[u]);
                        cp[i] = fma(t[x][i], rx, cp[i]);
                    }
                });
                const double rs = row_sums(rp, tj);
                if ((tj & 3) == 0) rowpart[par][16 * (x0 + (tj >> 2)) + ti] = rs;
            });
#pragma unroll
            for (int i = 0; i < N; i += 4) {
                if (2 * i + 7 < live) continue;
                const double cs = add_rows(add_halves(cp[i], cp[i + 2]), add_halves(cp[i + 1], cp[i + 3]));
                if (i + g < N) colpart[quarter][16 * (2 * (i + g) + par) + tj] = cs;
            }
        }
        __syncthreads();
        if (wave < NT / 2) {
            const int e = 32 * wave + (lane & 31), hh = lane >> 5;
            const double s = (colpart[2 * hh][e] + colpart[2 * hh + 1][e]) + rowpart[hh][e];
            const double p = add_halves(s, s);
            if (hh == 0) pbuf[e] = e > k ? p : 0.0;  // rows that are done
        }
        __syncthreads();
        const double beta = betas[k & 1];
        double kk, cw[N], rw = pbuf[16 * row_lane + ti];
#pragma unroll
        for (int i = 0; i < N; ++i) cw[i] = pbuf[16 * (2 * i + par) + tj];
        {
            double lv[Q], lp[Q], dot = 0.0;
            const double vc = v[k + 1], pc = pbuf[k + 1], v1 = v[k + 2], p1 = pbuf[k + 2];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                lv[q] = v[lane + 64 * q];
                lp[q] = pbuf[lane + 64 * q];
                dot = fma(lp[q], lv[q], dot);
            }
            kk = 0.5 * beta * (beta * wave_sum(dot));  // (beta^2 may overflow)
            if (wave == 0) {  // the others wait for it: ahead of the wavefront beside it on the SIMD
                __builtin_amdgcn_s_setprio(3);
#pragma unroll
                for (int q = 0; q < Q; ++q) lp[q] = fma(beta, lp[q], -kk * lv[q]);
                reflect(k + 1, lv, lp, vc, fma(beta, pc, -kk * vc), v1, fma(beta, p1, -kk * v1));
            }
        }
        {
            // (row k + 1 is on its way through arow, but behind the last step the tail takes it from the tiles)
            const int live = min(k + 2, stop) >> 4;
#pragma unroll
            for (int i = 0; i < N; ++i) cw[i] = fma(beta, cw[i], -kk * cv[i]);
            rw = fma(beta, rw, -kk * rv);
            unrolled<NT / 4>([&](auto bc) {
                constexpr int x0 = 4 * decltype(bc)::value;
                if (x0 + 3 < live) return;
                unrolled<4>([&](auto uc) {
                    constexpr int x = x0 + decltype(uc)::value;
                    const double rx = row_bcast<x>(rv), wx = row_bcast<x>(rw);
#pragma unroll
                    for (int i = x / 2; i < N; ++i) t[x][i] = fma(-rx, cw[i], fma(-wx, cv[i], t[x][i]));
                });
                unrolled<4>([&](auto uc) {
                    if (x0 + decltype(uc)::value == live)
                        keep_row(std::integral_constant<int, x0 + decltype(uc)::value>(), k + 2);
                });
            });
        }
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
    }
    // what is left, rows `stop` and on, in one wavefront
#pragma unroll
    for (int x = 0; x < NT; ++x)
#pragma unroll
        for (int i = x / 2; i < N; ++i) {
            const int y = 2 * i + par, p = 16 * x + ti - stop, q = 16 * y + tj - stop;
            if (y >= x && p >= 0 && q >= 0 && p < kTail && q < kTail) {
                sm[p][q] = t[x][i];
                if (y > x) sm[q][p] = t[x][i];
            }
        }
    __syncthreads();
    if (wave == 0 && r > 0) {
        reduce64([&](int i, int j) { return sm[i][j]; }, r - stop, lane == 0 ? tri + stop : unused + lane, sm, lane);
        wave_sync();
        const Interval in = gershgorin(tri, r, lane);
        for (int i = lane; i < 16 * sturm_blocks(r) + 8; i += 64)
            tri_of(it)[i] = i < r ? sturm_term(ldexp(tri[i].x, in.ex), i > 0 ? ldexp(tri[i].y, in.ex) : 0.0)
                                  : sturm_fill();
        if (lane == 0) {
            bounds_of(it)[0] = in.lo;
            bounds_of(it)[1] = in.hi;
        }
    }
    if (tid == 0) bounds_of(it)[2] = r;
}

// Ranks up to kFusedRank: the reduction in one wavefront, then the eigenvalues in all four, in bounds first: the
// share is nearly always decided after a third of their rounds.  Bound by latency: at r = 32 the reduction 32 K
// clocks (1040 a step), the eigenvalues 12 K, 5 K around them (one lane to a row, v and w through the LDS and
// the sums one after the other: 74 K and 22 K).  Whole calls, us before | after: 512 x 8 14.9 | 9.7, 512 x 16 21.4 |
// 13.1, 2048 x 32 46.5 | 27.9, 2048 x 48 79.0 | 48.9, 2048 x 64 105.8 | 64.0.
template <int RC>  // columns held: 32 or 64
__global__ __launch_bounds__(kTT) void tridiag_small_kernel(FactorBatch batch, double tau) {
    __shared__ double sm[RC][RC + 1];
    __shared__ double2 tri[RC + kSturmPad], unused[64 + RC + kSturmPad];
    __shared__ double eig[64], eig_hi[64];
    __shared__ int order[64];
    const FactorItem it = batch.it[blockIdx.x];
    const int nchunks = it.nchunks;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t rr = (int64_t)it.r * it.r;
    if (it.r > RC || it.r <= RC / 2 * (RC > 32)) return;  // another kernel's
    constexpr int E = RC * RC / kTT;
    int from[E];
    double sum[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = (tid + kTT * e) / RC, y = (tid + kTT * e) % RC;
        from[e] = x <= y && y < it.r ? x * it.r + y : -1;
        sum[e] = 0.0;
    }
    if constexpr (RC <= 32)
        if (nchunks == 0) {  // the sums are left to this kernel
            __shared__ double gram[4][kSmallGramRank][kSmallGramRank + 1];
            for (int c = 0; kGramChunk * c < it.L; ++c) {
                small_gram(it, c, gram);
                __syncthreads();
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int x = (tid + kTT * e) / RC % kSmallGramRank, y = (tid + kTT * e) % RC % kSmallGramRank;
                    sum[e] += ((gram[0][x][y] + gram[1][x][y]) + gram[2][x][y]) + gram[3][x][y];
                }
                __syncthreads();
            }
        }
    // Chunk by chunk in order, kAhead requested at a time, with the sums' launch, us at two | four | eight:
    // 8192 x 32 31.5 | 30.5 | 30.6, 2048 x 8 12.7 | 12.3 | 13.0, 512 x 32 28.3 | 27.9 | 28.7; with 64 columns one | two |
    // four: 512 x 48 48.1 | 48.2 | 49.3, 2048 x 64 65.2 | 65.0 | 64.9, 8192 x 64 65.9 | 66.0 | 67.3.
    constexpr int kAhead = RC <= 32 ? 4 : 2;
    for (int c = 0; c < nchunks; c += kAhead) {
        double p[kAhead][E];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int e = 0; e < E; ++e)
                p[u][e] = it.part[(c + u < nchunks ? c + u : c) * rr + (from[e] < 0 ? 0 : from[e])];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int e = 0; e < E; ++e) sum[e] += c + u < nchunks ? p[u][e] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = (tid + kTT * e) / RC, y = (tid + kTT * e) % RC;
        const double v = from[e] < 0 ? 0.0 : sum[e];
        if (x <= y) {
            sm[x][y] = v;
            sm[y][x] = v;
        }
    }
    __syncthreads();
    const double diag = lane < it.r ? sm[lane % RC][lane % RC] : 0.0;
    if (__ballot(!(diag < __builtin_inf()))) {
        // A NaN in S: r' = 0.  Infinities alone: every column of S is infinite and the first one holds
        // every share, up to rank 31; at 32, as above, 0.
        bool nan = false;
        for (int j = 0; j < it.r; ++j) nan = nan || (lane < it.r && sm[lane % RC][j] != sm[lane % RC][j]);
        const int32_t k = __ballot(nan) != 0 || it.r >= 32 ? 0 : 1;
        if (tid == 0) *it.out = k;
        return;
    }
    // the rows that are not zero, as in tridiag_kernel (every wavefront writes the same)
    const bool on = diag != 0.0;
    const uint64_t mask = __ballot(on);
    if (on) order[__popcll(mask & ((1ull << lane) - 1))] = lane;
    const int r = __popcll(mask);
    __syncthreads();
    if (wave == 0 && r > 0) {
        double2 *to = lane == 0 ? tri : unused + lane;
        auto element = [&](int i, int j) { return sm[order[i]][order[j]]; };
        if constexpr (RC <= 32) reduce32(element, r, to, lane);
        else reduce64(element, r, to, sm, lane);
    }
    __syncthreads();
    if (r == 0) {  // nothing but zeros
        if (tid == 0) *it.out = 0;
        return;
    }
    const Interval in = gershgorin(tri, r, lane);
    __syncthreads();  // every wavefront has its interval
    if (tid < r)
        tri[tid] = sturm_term(ldexp(tri[tid].x, in.ex), tid > 0 ? ldexp(tri[tid].y, in.ex) : 0.0);
    else if (tid < 16 * sturm_blocks(r) + 8)
        tri[tid] = sturm_fill();
    __syncthreads();
    // as many lanes per eigenvalue as 256 threads have for r of them
    auto find = [&](auto gc) {
        constexpr int G = decltype(gc)::value;
        const int c = tid / G;
        using R = Rounds<G>;
        double lo = in.lo, hi = in.hi;
        const int nth = c < r ? c : r - 1;
        const bool mine = c < r && (lane & (G - 1)) == 0;
        narrow<G>(tri, r, nth, lo, hi, lane, R::kEarly);
        if (mine) {
            eig[c] = lo;
            eig_hi[c] = hi;
        }
        __syncthreads();
        const double l[1] = {eig[lane]}, h[1] = {eig_hi[lane]};
        const int k = decided(l, h, r, tau, lane);  // by every wavefront, from the same
        if (k >= 0) {
            if (tid == 0) *it.out = k;
            return true;
        }
        narrow<G>(tri, r, nth, lo, hi, lane, R::kAll - R::kEarly);
        __syncthreads();
        if (mine) eig[c] = eigenvalue(lo, hi);
        if (tid >= r && tid < 64) eig[tid] = 0.0;
        return false;
    };
    bool done;
    if (r <= 4) done = find(std::integral_constant<int, 64>());
    else if (r <= 8) done = find(std::integral_constant<int, 32>());
    else if (r <= 16) done = find(std::integral_constant<int, 16>());
    else if (RC <= 32 || r <= 32) done = find(std::integral_constant<int, 8>());
    else done = find(std::integral_constant<int, 4>());
    if (done) return;
    __syncthreads();
    if (wave == 0) {
        const int32_t k = count_share(eig, r, tau, lane);
        if (lane == 0) *it.out = k;
    }
}

// Ranks above kFusedRank: one wavefront per eigenvalue, 64 points a round.  All lanes read the same terms, through
// the scalar cache.  Bound by the instructions of the sequence, four a term, two wavefronts to some SIMDs: 6.4 us a
// round for seven matrices at r = 256.  (32 lanes per eigenvalue, one wavefront to a SIMD: 5.4 us, but how many
// lanes there are for one would then depend on the batch, and with it the last bit of an eigenvalue, which decides
// where tau falls on a whole number of equal ones.)  After kEarlyRounds, at 2^-29, the bounds nearly always tell
// already which sums hold the share (at four, 2^-23, one factor in ten would go on).
constexpr int kEarlyRounds = 5;
__global__ __launch_bounds__(256) void eigenvalue_bounds_kernel(FactorBatch batch) {
    const FactorItem it = batch.it[blockIdx.y];
    if (it.r <= kFusedRank) return;
    const int r = live_of(it);
    const int lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (c >= r) return;
    const double2 *__restrict__ tri = tri_of(it);
    double lo = bounds_of(it)[0], hi = bounds_of(it)[1];
    narrow<64>(tri, r, c, lo, hi, lane, kEarlyRounds);
    if (lane == 0) {
        low_of(it)[c] = lo;
        high_of(it)[c] = hi;
    }
}

// r' from those bounds, or else the eigenvalues to the end and r' by count_kernel (open_of: 1).
__global__ __launch_bounds__(256) void eigenvalues_kernel(FactorBatch batch, double tau) {
    const FactorItem it = batch.it[blockIdx.y];
    if (it.r <= kFusedRank) return;
    const int r = live_of(it);
    const int lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double *__restrict__ low = low_of(it), *__restrict__ high = high_of(it);
    constexpr int N = DLCX_MAX_RANK / 64;
    double l[N], h[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int e = 64 * q + lane < r ? 64 * q + lane : 0;
        l[q] = low[e];
        h[q] = high[e];
    }
    const int k = r > 0 ? decided(l, h, r, tau, lane) : -1;
    if (k < 0 && c < r) {
        const double2 *__restrict__ tri = tri_of(it);
        double lo = low[c], hi = high[c];
        narrow<64>(tri, r, c, lo, hi, lane, Rounds<64>::kAll - kEarlyRounds);
        if (lane == 0) eig_of(it)[c] = eigenvalue(lo, hi);
    }
    // Behind all that is read: the table goes through the scalar cache as long as nothing is stored before it.
    if (c == 0 && lane == 0) {
        *open_of(it) = k < 0 ? 1.0 : 0.0;
        if (k >= 0) *it.out = k;
    }
}

__global__ __launch_bounds__(64) void count_kernel(FactorBatch batch, double tau) {
    __shared__ double eig[DLCX_MAX_RANK];
    const FactorItem it = batch.it[blockIdx.x];
    if (it.r <= kFusedRank || *open_of(it) == 0.0) return;
    const int r = live_of(it);
    for (int c = threadIdx.x; c < DLCX_MAX_RANK; c += 64) eig[c] = c < r ? eig_of(it)[c] : 0.0;
    __syncthreads();
    const int32_t k = count_share(eig, r, tau, threadIdx.x);
    if (threadIdx.x == 0) *it.out = k;
}

// doubles of the partial sums, whole pairs: what follows them is read and written in pairs
static size_t partial_doubles(int64_t L, int r) { return ((size_t)gram_chunks(L) * r * r + 1) & ~(size_t)1; }

size_t effrank_workspace_bytes(int64_t L, int r) {
    const size_t re = (size_t)((r + 1) & ~1);
    return a256x((partial_doubles(L, r) + re * re) * sizeof(double));
}

void effrank_item(FactorItem *it, const float *q_bar, int64_t L, int r, int32_t *out,
                  void *workspace) {
    it->f = const_cast<float *>(q_bar);  // only read
    it->L = L;
    it->r = r;
    it->nchunks = gram_chunks(L);
    it->part = reinterpret_cast<double *>(workspace);
    it->g = it->part + partial_doubles(L, r);
    it->w = nullptr;
    it->out = out;
}

int launch_effective_rank_batch(const FactorBatch &batch, double tau, hipStream_t st) {
    if (batch.n == 0) return DLCX_OK;
    FactorBatch summed = batch;  // the same factors with their Gram sums in one chunk where that pays, or none
    bool small = true;
    for (int i = 0; i < batch.n; ++i)
        small = small && batch.it[i].r <= kSmallGramRank && batch.it[i].L <= kSmallGramLength;
    if (small) {
        for (int i = 0; i < batch.n; ++i) summed.it[i].nchunks = 0;
    } else {
        int rc = launch_gram_partials_batch(batch, &summed, 0, st);
        if (rc != DLCX_OK) return rc;
    }
    int rmax = 0, rmin = DLCX_MAX_RANK;
    bool rmid = false;
    for (int i = 0; i < batch.n; ++i) {
        const int r = batch.it[i].r;
        rmax = r > rmax ? r : rmax;
        rmin = r < rmin ? r : rmin;
        rmid = rmid || (r > 32 && r <= kFusedRank);
    }
    Timed timed(KID_EFF_RANK, st);
    const dim3 grid((unsigned)batch.n), threads(kTT);
    // each kernel leaves the factors of another rank class alone
    if (rmin <= 32) hipLaunchKernelGGL(tridiag_small_kernel<32>, grid, threads, 0, st, summed, tau);
    if (rmid) hipLaunchKernelGGL(tridiag_small_kernel<64>, grid, threads, 0, st, summed, tau);
    if (rmax > kFusedRank) {
        if (rmax <= 128)
            hipLaunchKernelGGL(tridiag_kernel<8>, grid, dim3(kTri), 0, st, summed);
        else if (rmax <= 192)
            hipLaunchKernelGGL(tridiag_kernel<12>, grid, dim3(kTri), 0, st, summed);
        else
            hipLaunchKernelGGL(tridiag_kernel<16>, grid, dim3(kTri), 0, st, summed);
        const dim3 each((unsigned)ceil_div(rmax, 4), (unsigned)batch.n);
        hipLaunchKernelGGL(eigenvalue_bounds_kernel, each, dim3(256), 0, st, summed);
        hipLaunchKernelGGL(eigenvalues_kernel, each, dim3(256), 0, st, summed, tau);
        hipLaunchKernelGGL(count_kernel, grid, dim3(64), 0, st, summed, tau);
    }
    return check_launch("effective_rank");
}

int launch_effective_rank(int64_t L, int r, const float *q_bar, double tau, int32_t *rprime_dev,
                          void *workspace, hipStream_t st) {
    FactorBatch b;
    b.n = 1;
    effrank_item(&b.it[0], q_bar, L, r, rprime_dev, workspace);
    return launch_effective_rank_batch(b, tau, st);
}

}  // namespace dlcx
