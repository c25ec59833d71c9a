// Pair distances, radius bins and correlation sums (Sec. 2.1, eqs. eCDF and
// CIL) on gfx950.
//
// Canonical squared distance of two patterns a, b of length d:
//   d_k = fl64(a_k - b_k)  (inputs converted to double),
//   D   = RN64(sum_k d_k^2)   -- the exact sum, rounded once.
// Counting rule: a pair lies under radius R_m when D < fl(R_m * R_m).
//
// Pipeline for every pair statistic:
//   1. fast pass -> FP64 partials P[split][i][j] over K ranges:
//      FP64 sets: direct differences, P = sum d_k^2 over the range (k_dist_partial);
//      FP32 sets: split-bf16x3 Gram on the matrix cores (gram.hip).
//   2. k_classify sums the partials in a fixed order into D~ and its rigorous
//      bound eps (direct: all terms are non-negative, so any summation order
//      is within gamma_{d+S} D~ of the exact sum, and eps = (d + S + 4)
//      2^-53 1.01 D~; Gram: the bound derived in gram.hip), then bins the pair
//      or, when |D~ - fl(R_m^2)| <= eps for some m, puts it on a re-check list.
//   3. k_canonical recomputes the listed pairs canonically; every count is exact.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "cil_internal.hpp"
#include "dd_round.hpp"
#include "distance_async.hpp"
#include "radii_dd.hpp"

// The error-free transformations below (two-sum, exact squares split by an
// FMA) are only exact if no product is fused into a later sum: contraction
// off for this file; the fused multiply-adds that are wanted are explicit.
#pragma clang fp contract(off)

namespace cil {

// gram.hip
struct GramWork {
    __bf16 *Ah, *Al, *Bh, *Bl;
    double *na, *nb;
    float *c;
    long long dimP;
};
int gram_prepare(const float *, long long, const float *, long long, long long, GramWork *, hipStream_t);
long long gram_splits(long long, long long, long long);
int gram_partials(const GramWork &, long long, long long, long long, long long, double *, hipStream_t);

constexpr int TILE = 64;       // pairs per tile side (direct pass)
constexpr int KC = 16;         // k-chunk staged in LDS
constexpr int MAX_M = 255;

__device__ __forceinline__ double ld(const double *p) { return *p; }
__device__ __forceinline__ double ld(const float *p) { return (double)*p; }

// ------------------------------------------------------------ direct pass
// One 64 x 64 tile of pairs and one K range per block of 256 threads; thread
// (ty, tx) owns rows ty + 16 i and columns tx + 16 j, i, j < 4.
template <typename T>
__global__ __launch_bounds__(256) void k_dist_partial(const T *A, long long nA, const T *B, long long nB,
                                                      long long dim, long long ksplit, double *P)
{
    __shared__ double sA[TILE][KC + 1];
    __shared__ double sB[TILE][KC + 1];
    const int tid = threadIdx.x;
    const int tx = tid % 16, ty = tid / 16;
    const long long i0 = (long long)blockIdx.y * TILE, j0 = (long long)blockIdx.x * TILE;
    const long long kb = (long long)blockIdx.z * ksplit;
    const long long ke = kb + ksplit < dim ? kb + ksplit : dim;
    double acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
    for (long long k0 = kb; k0 < ke; k0 += KC) {
        __syncthreads();
        for (int e = tid; e < TILE * KC; e += 256) {
            const int r = e / KC, kk = e % KC;
            const long long k = k0 + kk;
            const long long ia = i0 + r, jb = j0 + r;
            sA[r][kk] = (ia < nA && k < ke) ? ld(A + ia * dim + k) : 0.0;
            sB[r][kk] = (jb < nB && k < ke) ? ld(B + jb * dim + k) : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            double a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = sA[ty + 16 * i][kk];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = sB[tx + 16 * j][kk];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double dlt = a[i] - b[j];
                    acc[i][j] = fma(dlt, dlt, acc[i][j]);
                }
        }
    }
    double *Ps = P + (long long)blockIdx.z * nA * nB;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const long long ia = i0 + ty + 16 * i, jb = j0 + tx + 16 * j;
            if (ia < nA && jb < nB) Ps[ia * nB + jb] = acc[i][j];
        }
}

// ---------------------------------------------------------------- classify
enum { MODE_BINS = 0, MODE_RANGE1 = 1, MODE_RANGE2 = 2, MODE_DUMP = 3 };

struct ClassifyArgs {
    const double *P;            // partials [S][nA][nB]
    int S;
    int gram;                   // 0: direct partials of D, 1: Gram partials
    const double *na, *nb;      // Gram: |a^|^2, |b^|^2
    double eps_rel;             // direct
    double eG;                  // Gram: eG / (|a'||b'|)
    double e1;                  // Gram: split error per element
    int mode;
    int exclude_diag;
    const double *thr;          // bins: [M]
    double thr_slack;           // bins: also list the pairs within thr_slack thr of a threshold
    int M;
    unsigned long long *hist;   // bins: [M+1]
    uint8_t *bins;              // bins: [nA][nB] or null
    int2 *list;                 // re-check / candidate list
    unsigned long long *nlist;
    long long cap;
    unsigned long long *minmax; // range: [min(D~+eps) bits, max(D~-eps) bits]
    unsigned long long *flag;   // range: set when a distance is not finite
    double *reduced;            // range pass 1: the summed partials of every pair, or null
    double *dump_d, *dump_eps;  // dump
};

__device__ __forceinline__ void approx_pair(const ClassifyArgs &c, long long i, long long j, long long nA,
                                            long long nB, double &D, double &eps)
{
    double s = 0.0;
    const double *pp = c.P + i * nB + j;
    const long long ps = nA * nB;
    int k = 0;
    for (; k + 8 <= c.S; k += 8) {               // eight loads in flight, added in order
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = pp[(k + u) * ps];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; k < c.S; ++k) s += pp[k * ps];
    // the sum of the partials, for the later passes (0 + s is s exactly, so
    // they see the same D~ from one partial)
    if (c.reduced) c.reduced[i * nB + j] = s;
    if (!c.gram) {
        D = s;
        eps = c.eps_rel * s;
        return;
    }
    const double na = c.na[i], nb = c.nb[j];
    D = na + nb - 2.0 * s;
    const double ra = sqrt(na), rb = sqrt(nb);
    const double Sg = ra + rb;
    const double eG = c.eG * ra * rb;
    const double Dp = D > 0.0 ? D : 0.0;
    const double u = 0x1p-53;
    const double bound = 2.0 * eG + 2.0 * c.e1 * Sg * (sqrt(Dp + 2.0 * eG) + c.e1 * Sg) + c.e1 * c.e1 * Sg * Sg +
                         8.0 * u * (na + nb + Dp) + u * Dp;
    eps = 2.0 * bound;
}

// One pair per lane and turn, the pairs in order over the whole grid; a lane's
// next pair is found by steps of (rows, columns), without a division.  At most
// 1024 workgroups of 512: the closing atomics all go to a few addresses, and
// with 4096 of 256 they took longer than the pass.  2048 x 2048 pairs (four partial
// planes): first range pass 69 us, second 29, bins against 32 thresholds
// 51 (121, 31, 98 so, and with a division per pair and every threshold compared).
constexpr int CLS = 512;
template <int MODE>
__global__ __launch_bounds__(CLS) void k_classify(ClassifyArgs c, long long nA, long long nB)
{
    __shared__ unsigned int hist[MAX_M + 1];
    __shared__ double sthr[MAX_M];
    __shared__ unsigned long long rlo[CLS / 64], rhi[CLS / 64];
    __shared__ int rbad[CLS / 64];
    const int tid = threadIdx.x;
    int top = 1;                                  // the power of two above M / 2: first step of the threshold search
    if constexpr (MODE == MODE_BINS) {
        for (int m = tid; m <= c.M; m += CLS) hist[m] = 0;
        for (int m = tid; m < c.M; m += CLS) sthr[m] = c.thr[m];
        while (2 * top <= c.M) top *= 2;
        __syncthreads();
    }
    const long long n = nA * nB;
    unsigned long long lo = ~0ull, hi = 0ull;     // RANGE1: bounds over this thread's pairs
    int bad = 0;
    // grid-stride over the pairs (the grid is capped, so per-block reductions stay few)
    const long long stride = (long long)gridDim.x * CLS, di = stride / nB, dj = stride % nB;
    long long e = (long long)blockIdx.x * CLS + tid, i = e / nB, j = e % nB;
    for (; e < n; e += stride, i += di, j += dj) {
        if (j >= nB) {
            j -= nB;
            ++i;
        }
        if (c.exclude_diag && i == j && !c.reduced) continue;
        double D, eps;
        approx_pair(c, i, j, nA, nB, D, eps);
        if (c.exclude_diag && i == j) continue;     // summed for the later passes, not part of the range
        const bool finite = isfinite(D) && isfinite(eps);
        if constexpr (MODE == MODE_BINS) {
            // the thresholds fall: bin = how many exceed D, by bisection; the
            // nearest on either side decides whether one is too close
            int bin = 0;
            for (int w = top; w > 0; w >>= 1)
                if (bin + w <= c.M && D < sthr[bin + w - 1]) bin += w;
            const double above = sthr[bin > 0 ? bin - 1 : 0], below = sthr[bin < c.M ? bin : c.M - 1];
            const bool amb = !finite || fabs(D - above) <= eps + c.thr_slack * above ||
                             fabs(D - below) <= eps + c.thr_slack * below;
            if (amb) {
                const unsigned long long slot = atomicAdd(c.nlist, 1ull);
                if ((long long)slot < c.cap) c.list[slot] = make_int2((int)i, (int)j);
            } else {
                atomicAdd(&hist[bin], 1u);
                if (c.bins) c.bins[i * nB + j] = (uint8_t)bin;
            }
        } else if constexpr (MODE == MODE_RANGE1) {
            // the bit patterns of non-negative doubles order as the values
            if (!finite) {
                bad = 1;
            } else {
                const unsigned long long l = (unsigned long long)__double_as_longlong(D + eps);
                const unsigned long long h = (unsigned long long)__double_as_longlong(fmax(D - eps, 0.0));
                lo = l < lo ? l : lo;
                hi = h > hi ? h : hi;
            }
        } else if constexpr (MODE == MODE_RANGE2) {
            const double mnub = __longlong_as_double((long long)c.minmax[0]);
            const double mxlb = __longlong_as_double((long long)c.minmax[1]);
            if (D - eps <= mnub || D + eps >= mxlb) {
                const unsigned long long slot = atomicAdd(c.nlist, 1ull);
                if ((long long)slot < c.cap) c.list[slot] = make_int2((int)i, (int)j);
            }
        } else {
            c.dump_d[e] = D;
            c.dump_eps[e] = eps;
        }
    }
    if constexpr (MODE == MODE_BINS) {
        __syncthreads();
        for (int m = tid; m <= c.M; m += CLS)
            if (hist[m]) atomicAdd(&c.hist[m], (unsigned long long)hist[m]);
    } else if constexpr (MODE == MODE_RANGE1) {
        // wavefront, then workgroup, then one atomic per workgroup
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long l2 = __shfl_xor(lo, o, 64), h2 = __shfl_xor(hi, o, 64);
            lo = l2 < lo ? l2 : lo;
            hi = h2 > hi ? h2 : hi;
            bad |= __shfl_xor(bad, o, 64);
        }
        if ((tid & 63) == 0) {
            rlo[tid >> 6] = lo;
            rhi[tid >> 6] = hi;
            rbad[tid >> 6] = bad;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < CLS / 64; ++w) {
                lo = rlo[w] < lo ? rlo[w] : lo;
                hi = rhi[w] > hi ? rhi[w] : hi;
                bad |= rbad[w];
            }
            if (bad) atomicOr(c.flag, 1ull);          // a non-finite distance
            // (no atomic where one before it has done as much)
            if (lo < __hip_atomic_load(&c.minmax[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&c.minmax[0], lo);
            if (hi > __hip_atomic_load(&c.minmax[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&c.minmax[1], hi);
        }
    }
}

// ---------------------------------------------------------------- canonical
// Double-double accumulation of the exact squares, one wavefront per pair (or
// sixteen, when few pairs are re-checked), then a certified rounding: with the
// relative error bound delta, RN(sum) = RN(hi + lo) whenever the interval
// [S - delta S, S + delta S] holds no rounding boundary.  Where it holds one
// (an exact tie, above all) the pair is summed again with a record of whether
// any rounding lost bits: if none did, hi + lo is the exact sum and the
// hardware's RN(hi + lo) is the correctly rounded value, ties included.  If
// that does not decide it either (or when forced) the wavefront recomputes
// the sum exactly: each lane builds a non-overlapping expansion of its terms
// (Shewchuk's exact summation), lane 0 merges the 64 expansions and rounds
// once, half to even.

// (hi, lo) += (bh, bl); inexact |= some rounding lost bits
__device__ __forceinline__ void dd_add_t(double &hi, double &lo, double bh, double bl, int &inexact)
{
    double s, e, t, et, u, eu;
    two_sum(hi, bh, s, e);
    two_sum(lo, bl, t, et);
    two_sum(e, t, u, eu);
    inexact |= (et != 0.0) | (eu != 0.0);
    hi = s + u;
    lo = u - (hi - s);
}

// (hi, lo) += d^2 without tracking: hi by an exact two-sum, everything it
// loses into lo, which is rounded.  Eleven FP64 operations a term against
// twenty-five of dd_add_t.  After k terms of a non-negative sum S the error is
// at most (2 k^2 + 2 k) 2^-106 S: |lo| stays below 2 k 2^-53 S, and each of the
// k updates rounds lo and the term added to it once.
__device__ __forceinline__ void dd_square(double &hi, double &lo, double d)
{
    const double p = d * d;
    double s, e;
    two_sum(hi, p, s, e);
    hi = s;
    lo += e + fma(d, d, -p);
}

// Relative error bound of a sum of per-lane dd_square accumulations of k terms
// each, joined by `joins` levels of double-double additions.
__device__ __forceinline__ double dd_delta(double k, double joins)
{
    return (4.0 * k * k + 4.0 * k + 64.0 * (joins + 1.0)) * 0x1p-106;
}

// S += d^2 for S that starts at a power of two top >= every d^2: t = fl(S + d^2)
// and t - S are then exact in what they keep, and what they lose is one more
// fused operation, five in all.  After k terms with the sum s, S - top + lo is
// within (k^2 + k) 2^-106 (top + s) of it: every rest is at most 2^-53 (top + s),
// rounded once itself and once a term in lo.
__device__ __forceinline__ void top_square(double &S, double &lo, double d)
{
    const double t = fma(d, d, S);
    lo += fma(d, d, -(t - S));
    S = t;
}

constexpr int EXP_CAP = 64;     // a non-overlapping expansion of doubles has < 40 parts

__device__ __forceinline__ void exp_add(double (&part)[EXP_CAP], int &np, double x)
{
    int k = 0;
    for (int i = 0; i < np; ++i) {
        double y = part[i];
        if (fabs(x) < fabs(y)) {
            const double t = x;
            x = y;
            y = t;
        }
        const double hi = x + y;
        const double lo = y - (hi - x);
        if (lo != 0.0) part[k++] = lo;
        x = hi;
    }
    part[k++] = x;
    np = k;
}

__device__ __forceinline__ double exp_round(const double (&part)[EXP_CAP], int np)
{
    if (np == 0) return 0.0;
    int m = np;
    double hi = part[--m], lo = 0.0;
    while (m > 0) {
        const double x = hi, y = part[--m];
        hi = x + y;
        lo = y - (hi - x);
        if (lo != 0.0) break;
    }
    if (m > 0 && ((lo < 0.0 && part[m - 1] < 0.0) || (lo > 0.0 && part[m - 1] > 0.0))) {
        const double y = lo * 2.0, x = hi + y;
        if (y == x - hi) hi = x;
    }
    return hi;
}

// Exact sum over the wavefront (all 64 lanes call it); result valid in lane 0.
template <typename T>
__device__ double exact_d2_wave(const T *a, const T *b, long long dim, int lane)
{
    double part[EXP_CAP];
    int np = 0;
    for (long long k = lane; k < dim; k += 64) {
        const double d = ld(a + k) - ld(b + k);
        const double p = d * d;
        const double e = fma(d, d, -p);
        exp_add(part, np, p);
        if (e != 0.0) exp_add(part, np, e);
    }
    int maxm = np;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) maxm = max(maxm, __shfl_xor(maxm, o, 64));
    for (int src = 1; src < 64; ++src) {
        for (int c = 0; c < maxm; ++c) {
            const double mine = c < np ? part[c] : 0.0;
            const double v = __shfl(mine, src, 64);
            if (lane == 0 && v != 0.0) exp_add(part, np, v);
        }
    }
    return lane == 0 ? exp_round(part, np) : 0.0;
}

// The sum over k = from, from + stride, ... of one wavefront's lanes with a record of
// lost bits, joined over the lanes.
template <typename T>
__device__ __forceinline__ void tracked_sum(const T *a, const T *b, long long dim, long long from, long long stride,
                                            double &hi, double &lo, int &inexact)
{
    hi = lo = 0.0;
    inexact = 0;
    for (long long k = from; k < dim; k += stride) {
        const double d = ld(a + k) - ld(b + k);
        const double p = d * d;
        dd_add_t(hi, lo, p, fma(d, d, -p), inexact);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double oh = __shfl_xor(hi, off, 64), ol = __shfl_xor(lo, off, 64);
        dd_add_t(hi, lo, oh, ol, inexact);
        inexact |= __shfl_xor(inexact, off, 64);
    }
}

// The rounding of a tracked sum, by one wavefront: as it is where no bit was lost or
// the certificate holds, else by the exact summation.  (Lane 0's value counts.)
template <typename T>
__device__ __attribute__((noinline)) double tracked_round(const T *a, const T *b, long long dim, int lane, double hi,
                                                          double lo, int inexact, int force_exact,
                                                          unsigned long long *nexact)
{
    double D;
    int certain = dd_certain(hi, lo, (double)(dim + 65 * 17) * 0x1p-100, D);   // relative error bound
    certain = isfinite(D) && (certain || !inexact);
    certain = __shfl(certain, 0, 64);
    D = __shfl(D, 0, 64);
    if (!certain || force_exact) {
        D = exact_d2_wave(a, b, dim, lane);
        if (lane == 0) atomicAdd(nexact, 1ull);
    }
    return D;
}

// The pairs the untracked sum cannot certify, by one wavefront: ties, and one in
// 2^30 or so.  (Of FP32 sets one in some tens: the squares' last bits lie few
// places below their sum's, so that many sums end on a rounding boundary.)
template <typename T>
__device__ __attribute__((noinline)) double canonical_tracked(const T *a, const T *b, long long dim, int lane,
                                                              int force_exact, unsigned long long *nexact)
{
    double hi, lo;
    int inexact;
    tracked_sum(a, b, dim, lane, 64, hi, lo, inexact);
    return tracked_round(a, b, dim, lane, hi, lo, inexact, force_exact, nexact);
}

struct CanonOut {
    // pair source: either an int2 list (recheck) or two index arrays
    const int2 *pairs;
    const unsigned long long *npairs_dev;   // count for the list (clamped to cap)
    long long cap;
    long long first;            // list mode: the launch covers pairs first, first + 1, ...
    long long stride;           // list mode: > 0 loops each wave (WPP 1) or block over w, w + stride, ...
    const long long *ia, *jb;
    long long npairs;
    long long nA;               // index bounds for the ia/jb source
    int *bad;                   // set when an ia/jb index is out of range
    // sinks
    double *d2;                 // per pair, or null
    unsigned long long *range_mm;   // or null: [0] min, [1] max of the pairs' D (bits of non-negative doubles)
    const double *thr;
    int M;
    unsigned long long *hist;   // or null
    uint8_t *bins;              // or null
    double win_rel;             // with win_hits: bit m set when a pair lies within win_rel thr[m] of thr[m]
    unsigned long long *win_hits;
    long long nB;
    unsigned long long *nexact;
    int force_exact;
    const int *only_if;         // or null: the launch leaves at once where this is 0
};

// WPP wavefronts per pair: 1 (four pairs per 256-thread block; many pairs, the
// pass is bandwidth-bound), 4 or 16 (one pair per block; fewer pairs,
// latency-bound).  The certified rounding makes the result independent of
// the summation order, so both give the same doubles.
template <typename T, int WPP>
__device__ __forceinline__ void canonical_pair(const T *A, const T *B, long long dim, const CanonOut &o, long long w,
                                               int lane, int sub);

template <typename T, int WPP>
__global__ __launch_bounds__(WPP == 1 ? 256 : 64 * WPP) void k_canonical(const T *A, const T *B, long long dim,
                                                                         CanonOut o)
{
    if (o.only_if && !*o.only_if) return;
    const int lane = threadIdx.x & 63;
    const int sub = WPP == 1 ? 0 : threadIdx.x / 64;
    // list mode: the grid may be sized before the list count is known (an
    // upper bound); waves past the count leave at once, or with a stride
    // (the grid's pair slots) each wave or block takes every stride-th pair
    const long long w = (WPP == 1 ? (long long)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64
                                  : (long long)blockIdx.x) + (o.pairs ? o.first : 0);
    const long long np = o.pairs ? (long long)min((unsigned long long)o.cap, *o.npairs_dev) : o.npairs;
    if (o.pairs && o.stride > 0) {       // the trip count is uniform over a block
        for (long long v = w; v < np; v += o.stride) {
            canonical_pair<T, WPP>(A, B, dim, o, v, lane, sub);
            if constexpr (WPP > 1) __syncthreads();   // wave 0 is done with the pair's partials
        }
        return;
    }
    if (w >= np) return;
    canonical_pair<T, WPP>(A, B, dim, o, w, lane, sub);
}

// The canonical squared distance of pair w (of the list or the index arrays)
// and its sinks, by one wave (WPP 1) or the block's WPP waves.
template <typename T, int WPP>
__device__ __forceinline__ void canonical_pair(const T *A, const T *B, long long dim, const CanonOut &o, long long w,
                                               int lane, int sub)
{
    long long i, j;
    if (o.pairs) {
        i = o.pairs[w].x;
        j = o.pairs[w].y;
    } else {
        i = o.ia[w];
        j = o.jb[w];
        if (i < 0 || i >= o.nA || j < 0 || j >= o.nB) {
            if (lane == 0) {
                if (o.d2) o.d2[w] = NAN;
                atomicOr(o.bad, 1);
            }
            return;
        }
    }
    const T *a = A + i * dim;
    const T *b = B + j * dim;
    double hi = 0.0, lo = 0.0;
    constexpr long long STR = 64LL * WPP;
    long long k = lane + 64LL * sub;
    for (; k + 3 * STR < dim; k += 4 * STR) {            // four strides' loads in flight
        double da[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) da[u] = ld(a + k + u * STR) - ld(b + k + u * STR);
#pragma unroll
        for (int u = 0; u < 4; ++u) dd_square(hi, lo, da[u]);
    }
    for (; k < dim; k += STR) dd_square(hi, lo, ld(a + k) - ld(b + k));
    int unused = 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double oh = __shfl_xor(hi, off, 64), ol = __shfl_xor(lo, off, 64);
        dd_add_t(hi, lo, oh, ol, unused);
    }
    double D;
    const double delta = dd_delta((double)((dim + STR - 1) / STR), 6 + WPP);
    if constexpr (WPP > 1) {      // combine the pair's wavefronts; wavefront 0 finishes
        __shared__ double phi[WPP], plo[WPP];
        __shared__ int pin[WPP], again;
        if (lane == 0) {
            phi[sub] = hi;
            plo[sub] = lo;
        }
        __syncthreads();
        if (sub == 0) {
            for (int v = 1; v < WPP; ++v) dd_add_t(hi, lo, phi[v], plo[v], unused);
            const bool certain = dd_certain(hi, lo, delta, D);
            if (lane == 0) again = !certain || o.force_exact;
            D = __shfl(D, 0, 64);
        }
        __syncthreads();
        if (again) {              // uniform: all of them sum it again (678 pairs of d = 8192, FP32: 77 us by one alone, 42 so)
            int inexact;
            tracked_sum(a, b, dim, lane + 64LL * sub, STR, hi, lo, inexact);
            if (lane == 0) {
                phi[sub] = hi;
                plo[sub] = lo;
                pin[sub] = inexact;
            }
            __syncthreads();
            if (sub == 0) {
                for (int v = 1; v < WPP; ++v) {
                    dd_add_t(hi, lo, phi[v], plo[v], inexact);
                    inexact |= pin[v];
                }
                D = tracked_round(a, b, dim, lane, hi, lo, inexact, o.force_exact, o.nexact);
            }
        }
        if (sub != 0) return;
    } else {
        int certain = dd_certain(hi, lo, delta, D);
        certain = __shfl(certain, 0, 64);                // lane 0 decides for the wavefront
        D = __shfl(D, 0, 64);
        if (!certain || o.force_exact) D = canonical_tracked(a, b, dim, lane, o.force_exact, o.nexact);
    }
    if (lane == 0) {
        if (o.d2) o.d2[w] = D;
        if (o.range_mm) {       // non-negative doubles order as their bit patterns
            atomicMin(&o.range_mm[0], (unsigned long long)__double_as_longlong(D));
            atomicMax(&o.range_mm[1], (unsigned long long)__double_as_longlong(D));
        }
        if (o.hist) {
            int bin = 0;
            unsigned long long near = 0;
            for (int m = 0; m < o.M; ++m) {
                bin += (D < o.thr[m]);
                if (o.win_hits && fabs(D - o.thr[m]) <= o.win_rel * o.thr[m]) near |= 1ull << m;
            }
            atomicAdd(&o.hist[bin], 1ull);
            if (near) atomicOr(o.win_hits, near);
            if (o.bins) o.bins[i * o.nB + j] = (uint8_t)bin;
        }
    }
}

// A power of two above every |x| of the row (infinite if one is), at least 2^-460.
template <typename T>
__global__ __launch_bounds__(256) void k_row_tops(const T *A, long long nA, const T *B, long long dim, double *tops,
                                                  const int *only_if)
{
    __shared__ double part[4];
    if (only_if && *only_if) return;
    const long long i = blockIdx.x;
    const T *row = i < nA ? A + i * dim : B + (i - nA) * dim;
    T m = T(0);
    auto take = [&](T x) __attribute__((always_inline)) {
        const T v = x < T(0) ? -x : x;
        m = v > m ? v : m;
    };
    constexpr int W = 16 / sizeof(T);                    // 16-byte loads from the first aligned value on
    using V = T __attribute__((ext_vector_type(W)));
    const long long head = min(dim, (long long)(-(intptr_t)row & 15) / (long long)sizeof(T)), body = (dim - head) / W;
    const V *v = reinterpret_cast<const V *>(row + head);
    for (long long k = threadIdx.x; k < head; k += 256) take(row[k]);
    for (long long k = threadIdx.x; k < body; k += 1024) {
        V x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = v[min(k + 256 * u, body - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int w = 0; w < W; ++w) take(x[u][w]);
    }
    for (long long k = head + W * body + threadIdx.x; k < dim; k += 256) take(row[k]);
    double t = (double)m;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t = fmax(t, __shfl_xor(t, o, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        t = fmax(fmax(part[0], part[1]), fmax(part[2], part[3]));
        int ex = 0;
        if (isfinite(t)) (void)frexp(t, &ex);
        tops[i] = isfinite(t) ? ldexp(1.0, t > 0.0 ? max(ex, -460) : -460) : t;
    }
}

// A power of two >= every squared difference of two rows with these tops.
__device__ __forceinline__ double pair_top(double a, double b)
{
    const double m = 2.0 * fmax(a, b);
    return m * m;
}

// All pairs of two sets at once.  Nothing is listed, so rows can be shared: a
// wavefront takes RW x CW pairs, its lanes along k, and reads RW + CW values for
// RW CW terms where a wavefront per pair reads two for one; a block of four takes
// 4 RW x CW pairs, KW such groups split k between them.  2 x 8 pairs and KW = 2 for
// many pairs, 1 x 4 and KW = 4 for few.  Bound by FP64 issue: 62 500 pairs of d =
// 8192 in FP32 take 140 us with top_square (its power of two per pair from the
// rows' largest entries, k_row_tops), 247 with dd_square's eleven operations a
// term, 385 by a wavefront per pair.  The sums of a wavefront are reduced by
// halving: at each of log2(RW CW) levels a lane hands over half of its pairs and
// keeps the rest, then plainly.
// With `square` the columns are one of several sets (blockIdx.z, strideB elements
// apart) and the pairs those within the set, of which only j >= i are formed and
// written twice, followed by those of A's rows with it (rows nB, nB + 1, ... of
// d2).  blockIdx.x then counts the tiles that are formed, one after the other, so
// that every XCD gets its share of them (by rows and columns the eight XCDs, which
// take workgroups in turn, had 1 to 8 of 36 tiles each: 1430 us for 20 sets of 64
// patterns of d = 32768 and 8 rows, 1016 so; 520 with top_square).
template <typename T, int RW, int CW, int KW>
__global__ __launch_bounds__(256 * KW) __attribute__((amdgpu_waves_per_eu(4))) void k_canonical_grid(
    const T *A, const double *topA, long long nA, const T *B, const double *topB, long long nB, long long dim, double *d2,
    int square, long long strideB, const int *only_if, int force_exact, unsigned long long *nexact)
{
    constexpr int NP = RW * CW, TI = 4 * RW;
    static_assert(CW % TI == 0, "a block's rows lie within one column tile");
    __shared__ double part[KW > 1 ? KW - 1 : 1][4][NP][2];
    if (only_if && *only_if) return;                     // the list is not the grid of all pairs
    // the wavefront's numbers in scalars: the rows' addresses then take no lane registers
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3),
              kw = KW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
    const unsigned nct = (unsigned)((nB + CW - 1) / CW);
    unsigned bi = blockIdx.x / nct, bj = blockIdx.x % nct;
    bool within = false;
    if (square) {
        constexpr unsigned RT = CW / TI;                 // row tiles to a column tile
        const unsigned ntri = RT * nct * (nct + 1) / 2, t = blockIdx.x;
        within = t < ntri;
        if (within) {                                    // column tile bj holds the row tiles 0 .. RT (bj + 1) - 1
            bj = (unsigned)((sqrtf(8.0f * (t / RT) + 1.0f) - 1.0f) * 0.5f);
            while (RT * (bj + 1) * (bj + 2) / 2 <= t) ++bj;
            while (RT * bj * (bj + 1) / 2 > t) --bj;
            bi = t - RT * bj * (bj + 1) / 2;
        } else {
            bi = (t - ntri) / nct;
            bj = (t - ntri) % nct;
        }
        B += blockIdx.z * strideB;
        topB += blockIdx.z * nB;
        d2 += blockIdx.z * (nA + nB) * nB + (within ? 0 : nB * nB);
        if (within) {
            A = B;
            topA = topB;
            nA = nB;
        }
    }
    bi = __builtin_amdgcn_readfirstlane(bi);
    bj = __builtin_amdgcn_readfirstlane(bj);
    const long long i0 = (long long)bi * TI + RW * wv, j0 = (long long)bj * CW;
    const T *ra[RW], *rb[CW];
#pragma unroll
    for (int r = 0; r < RW; ++r) ra[r] = A + min(i0 + r, nA - 1) * dim;
#pragma unroll
    for (int q = 0; q < CW; ++q) rb[q] = B + min(j0 + q, nB - 1) * dim;
    double hi[NP], lo[NP];
    auto each_top = [&](auto &&f) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int q = 0; q < CW; ++q) f(r * CW + q, pair_top(topA[min(i0 + r, nA - 1)], topB[min(j0 + q, nB - 1)]));
    };
    each_top([&](int e, double top) {
        hi[e] = top;
        lo[e] = 0.0;
    });
    // Blocks start at different k and wrap round: rows are often a power of two
    // apart, and at one k they would all be on one L2 channel (62 500 pairs of d =
    // 8192 in FP32: 325 against 582 us).
    constexpr long long STR = 64LL * KW;
    const unsigned chunks = (unsigned)((dim + STR - 1) / STR);
    const unsigned turn = (bj * 5u + bi * 3u + blockIdx.z) * 7u % chunks * (unsigned)STR;
    auto sum_range = [&](unsigned from, unsigned to) __attribute__((always_inline)) {
        unsigned k = from + lane + 64u * kw;
        if (k >= to) return;
        T a[RW], b[CW];                                  // read one round ahead
        auto read = [&](unsigned at) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < RW; ++r) a[r] = at_byte(ra[r], at * (unsigned)sizeof(T));
#pragma unroll
            for (int q = 0; q < CW; ++q) b[q] = at_byte(rb[q], at * (unsigned)sizeof(T));
        };
        read(k);
        while (true) {
            double av[RW], bv[CW];
#pragma unroll
            for (int r = 0; r < RW; ++r) av[r] = (double)a[r];
#pragma unroll
            for (int q = 0; q < CW; ++q) bv[q] = (double)b[q];
            k += (unsigned)STR;
            const bool more = k < to;
            read(more ? k : k - (unsigned)STR);
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int q = 0; q < CW; ++q) top_square(hi[r * CW + q], lo[r * CW + q], av[r] - bv[q]);
            if (!more) break;
        }
    };
    for (int lap = 0; lap < 2; ++lap) sum_range(lap ? 0u : turn, lap ? turn : (unsigned)dim);
    each_top([&](int e, double top) { two_sum(hi[e] - top, lo[e], hi[e], lo[e]); });
    int unused = 0;
    int mine = 0;                                        // first of the pairs the lane keeps
#pragma unroll
    for (int half = NP / 2; half >= 1; half >>= 1) {
        const int off = 64 / NP * half;
        const bool up = (lane & off) != 0;
        mine += up ? half : 0;
#pragma unroll
        for (int e = 0; e < half; ++e) {
            const double sh = up ? hi[e] : hi[e + half], sl = up ? lo[e] : lo[e + half];
            double kh = up ? hi[e + half] : hi[e], kl = up ? lo[e + half] : lo[e];
            dd_add_t(kh, kl, __shfl_xor(sh, off, 64), __shfl_xor(sl, off, 64), unused);
            hi[e] = kh;
            lo[e] = kl;
        }
    }
#pragma unroll
    for (int off = 32 / NP; off >= 1; off >>= 1)
        dd_add_t(hi[0], lo[0], __shfl_xor(hi[0], off, 64), __shfl_xor(lo[0], off, 64), unused);
    if constexpr (KW > 1) {
        if (kw > 0 && (lane & (64 / NP - 1)) == 0) {
            part[kw - 1][wv][mine][0] = hi[0];
            part[kw - 1][wv][mine][1] = lo[0];
        }
        __syncthreads();
        if (kw > 0) return;
        for (int v = 0; v < KW - 1; ++v) dd_add_t(hi[0], lo[0], part[v][wv][mine][0], part[v][wv][mine][1], unused);
    }
    double D;
    const long long i = i0 + mine / CW, j = j0 + mine % CW;
    const double k = (double)((dim + STR - 1) / STR), u2 = 2.0 * (k * k + k) * 0x1p-106;
    bool certain = dd_certain(hi[0], lo[0], dd_delta(0.0, 6 + KW) + u2, D,
                              u2 * (double)STR * pair_top(topA[min(i, nA - 1)], topB[min(j, nB - 1)]));
    const bool wanted = (lane & (64 / NP - 1)) == 0 && i < nA && j < nB && (!within || j >= i);
    unsigned long long redo = __ballot(wanted && (!certain || force_exact));
    while (redo) {                                       // rare: the whole wavefront sums that pair again
        const int src = __ffsll((long long)redo) - 1;
        redo &= redo - 1;
        const long long ii = __shfl(i, src, 64), jj = __shfl(j, src, 64);
        const double v = canonical_tracked(A + ii * dim, B + jj * dim, dim, lane, force_exact, nexact);
        const double w = __shfl(v, 0, 64);
        if (lane == src) D = w;
    }
    if (wanted) {
        d2[i * nB + j] = D;
        if (within) d2[j * nB + i] = D;
    }
}

// *not_grid |= the list is not (0, 0), (0, 1), ..., row by row over nB columns.
__global__ __launch_bounds__(256) void k_list_is_grid(const long long *ia, const long long *jb, long long np,
                                                      long long nB, int *not_grid)
{
    const long long w = (long long)blockIdx.x * 256 + threadIdx.x;
    if (w < np && (ia[w] != w / nB || jb[w] != w % nB)) *not_grid = 1;
}

// ======================================================================
// Host side.

namespace {
thread_local long long t_pairs = 0, t_rechecked = 0, t_exact = 0;
int g_force_exact = 0;

struct DistScratch {
    double *thr = nullptr;
    unsigned long long *hist = nullptr;
    unsigned long long *nlist = nullptr;
    unsigned long long *nexact = nullptr;
    unsigned long long *minmax = nullptr;
    unsigned long long *flag = nullptr;
    unsigned long long *cmm = nullptr;      // canonical extremes of the range candidates (bits)
    RangeOut *ro = nullptr;
    int2 *list = nullptr;
    long long cap = 0;
};

int scratch(long long cap, DistScratch *s)
{
    void *p;
    CIL_TRY(ws_get(WS_DIST_MISC, 4096 + sizeof(double) * 512, &p));
    char *c = (char *)p;
    s->thr = (double *)c;                                   // 256 doubles
    s->hist = (unsigned long long *)(c + 2048);             // 256 counters
    s->nlist = (unsigned long long *)(c + 4096);
    s->nexact = s->nlist + 1;
    s->minmax = s->nlist + 2;
    s->flag = s->nlist + 4;
    s->cmm = s->nlist + 5;
    s->ro = (RangeOut *)(c + 4096 + 64);
    static_assert(4096 + 64 + sizeof(RangeOut) <= 4096 + sizeof(double) * 512, "range output fits the workspace");
    CIL_TRY(ws_get(WS_DIST_RECHECK, sizeof(int2) * (size_t)std::max<long long>(cap, 1), &p));
    s->list = (int2 *)p;
    s->cap = cap;
    return CIL_OK;
}

constexpr long long kGridPairs = 32768;     // pairs from which sixteen a wavefront leave two wavefronts a SIMD
constexpr long long kGridDim = 1ll << 29;      // rows of less than 4 GB: byte offsets of 32 bits

// Whether all nA nB pairs gain by shared rows: the tiles of 8 x 8 pairs must not
// be mostly padding, and the rows long enough for the sums to outweigh the rows'
// tops and two launches.  us, shared rows / wavefront per pair, FP32: 40000 x 1
// of d = 512 170 / 79; 20000 x 2 of 512 108 / 78, of 4096 282 / 221; 10000 x 4 of
// 2 71 / 59, of 64 64 / 59, of 512 75 / 76, of 4096 154 / 212; 7000 x 7 of 2 67 / 62,
// of 64 60 / 63; 256 x 256 of 2 70 / 70, of 64 58 / 71, of 4096 118 / 311.
// (k_row_tops takes a workgroup of 256 per row, of at most 2^32 threads.)
bool grid_gains(long long nA, long long nB, long long dim)
{
    const long long np = nA * nB, padded = (nA + 7) / 8 * 8 * ((nB + 7) / 8 * 8);
    return np >= kGridPairs && padded <= 2 * np && dim >= (padded <= np + np / 4 ? 32 : 512) && dim < kGridDim &&
           nA + nB < 1ll << 24;
}

// Launches waves for pairs co.first .. co.first + nwaves - 1 (in list mode
// nwaves may exceed the list: the surplus waves leave at once).  Few pairs of long
// rows take four or sixteen wavefronts each (re-checks of d = 2048, FP32: 30 pairs
// 15.6 us by four, 21.8 by one; 2740 52.8 and 64.6; of d = 512 one is as good).
template <typename T>
int run_canonical(const T *A, const T *B, long long dim, CanonOut &co, long long nwaves, hipStream_t st)
{
    if (nwaves <= 0) return CIL_OK;
    const ProfMark pm = prof_begin("k_canonical", st);
    if (nwaves < 2048 && dim >= 4096)
        hipLaunchKernelGGL((k_canonical<T, 16>), dim3((unsigned)nwaves), dim3(1024), 0, st, A, B, dim, co);
    else if ((nwaves < kGridPairs && dim >= 4096) || (nwaves <= 2048 && dim >= 1024))
        hipLaunchKernelGGL((k_canonical<T, 4>), dim3((unsigned)nwaves), dim3(256), 0, st, A, B, dim, co);
    else
        hipLaunchKernelGGL((k_canonical<T, 1>), dim3((unsigned)((nwaves + 3) / 4)), dim3(256), 0, st, A, B, dim, co);
    prof_end(pm, st);
    return check_launch("k_canonical");
}

// All pairs of A and B (sets = 0), or the square form for `sets` sets.
template <typename T, int RW, int CW, int KW>
int launch_canonical_grid(const T *A, long long nA, const T *B, long long nB, long long strideB, long long dim,
                          double *d2, int sets, const int *only_if, unsigned long long *nexact, hipStream_t st)
{
    const long long nct = (nB + CW - 1) / CW, nrt = (nA + 4 * RW - 1) / (4 * RW);
    const dim3 grid = sets ? dim3((unsigned)(CW / (4 * RW) * nct * (nct + 1) / 2 + nrt * nct), 1, (unsigned)sets)
                           : dim3((unsigned)(nct * nrt));
    const long long rows = nA + (sets ? sets : 1) * nB;
    double *tops;
    CIL_TRY(ws_get(WS_DIST_TOPS, sizeof(double) * rows, (void **)&tops));
    const ProfMark pm = prof_begin("k_canonical_grid", st);
    hipLaunchKernelGGL((k_row_tops<T>), dim3((unsigned)rows), dim3(256), 0, st, A, nA, B, dim, tops, only_if);
    hipLaunchKernelGGL((k_canonical_grid<T, RW, CW, KW>), grid, dim3(256 * KW), 0, st, A, (const double *)tops, nA, B,
                       (const double *)tops + nA, nB, dim, d2, sets > 0, strideB, only_if, g_force_exact, nexact);
    prof_end(pm, st);
    return check_launch("k_canonical_grid");
}
template <typename T>
int run_canonical_grid(const T *A, long long nA, const T *B, long long nB, long long strideB, long long dim, double *d2,
                       int sets, const int *only_if, unsigned long long *nexact, hipStream_t st)
{
    const long long pairs = sets ? sets * (nA + nB / 2) * nB : nA * nB;
    if (pairs >= kGridPairs)
        return launch_canonical_grid<T, 2, 8, 2>(A, nA, B, nB, strideB, dim, d2, sets, only_if, nexact, st);
    return launch_canonical_grid<T, 1, 4, 4>(A, nA, B, nB, strideB, dim, d2, sets, only_if, nexact, st);
}

struct Approx {
    ClassifyArgs c{};
};

// Re-check launches are sized before the host knows the list's length: an
// upper bound covers the usual case in the same stream pass, and only a
// longer list costs a second launch after the count is read back.
long long recheck_guess(long long dim) { return dim >= 4096 ? 256 : 2048; }

// FP64 sets: direct differences, split over K so the grid fills the chip.
int approx_pass(const double *A, long long nA, const double *B, long long nB, long long dim, Approx *ap,
                hipStream_t st)
{
    const long long tiles = ((nA + TILE - 1) / TILE) * ((nB + TILE - 1) / TILE);
    long long S = 1;
    while (tiles * S < 1024 && dim / (2 * S) >= 256) S *= 2;
    const long long ks = std::max<long long>(KC, (dim / S + KC - 1) / KC * KC);
    S = std::max<long long>(1, (dim + ks - 1) / ks);
    void *p;
    CIL_TRY(ws_get(WS_DIST_SAMPLE, sizeof(double) * (size_t)std::max<long long>(S * nA * nB, 1), &p));
    ap->c.P = (const double *)p;
    ap->c.S = (int)S;
    ap->c.gram = 0;
    ap->c.eps_rel = (double)(dim + S + 4) * 0x1p-53 * 1.01;
    if (nA * nB > 0) {
        dim3 grid((unsigned)((nB + TILE - 1) / TILE), (unsigned)((nA + TILE - 1) / TILE), (unsigned)S);
        const ProfMark pm = prof_begin("k_dist_partial", st);
        hipLaunchKernelGGL(k_dist_partial<double>, grid, dim3(256), 0, st, A, nA, B, nB, dim, ks, (double *)p);
        prof_end(pm, st);
        CIL_TRY(check_launch("k_dist_partial"));
    }
    return CIL_OK;
}

// FP32 sets: split-bf16x3 Gram on the matrix cores.
int approx_pass(const float *A, long long nA, const float *B, long long nB, long long dim, Approx *ap,
                hipStream_t st)
{
    GramWork g;
    CIL_TRY(gram_prepare(A, nA, B, nB, dim, &g, st));
    long long S = gram_splits(nA, nB, g.dimP);
    const long long ks = std::max<long long>(64, (g.dimP / S + 63) / 64 * 64);
    S = std::max<long long>(1, (g.dimP + ks - 1) / ks);
    void *p;
    CIL_TRY(ws_get(WS_DIST_SAMPLE, sizeof(double) * (size_t)std::max<long long>(S * nA * nB, 1), &p));
    ap->c.P = (const double *)p;
    ap->c.S = (int)S;
    ap->c.gram = 1;
    ap->c.na = g.na;
    ap->c.nb = g.nb;
    ap->c.eG = 3.0 * (double)gram_flush_interval() * 0x1p-24 + 0x1p-18 + 0x1p-40;
    ap->c.e1 = 0x1p-24 + 0x1p-18;
    if (nA * nB > 0) CIL_TRY(gram_partials(g, nA, nB, S, ks, (double *)p, st));
    return CIL_OK;
}

int classify(ClassifyArgs &c, long long nA, long long nB, hipStream_t st)
{
    const long long n = nA * nB;
    if (n <= 0) return CIL_OK;
    const long long blocks = std::min<long long>((n + CLS - 1) / CLS, 1024);
    static const char *const names[] = {"k_classify_bins", "k_classify_range1", "k_classify_range2", "k_classify_dump"};
    const ProfMark pm = prof_begin(names[c.mode], st);
    void (*const kernels[])(ClassifyArgs, long long, long long) = {k_classify<MODE_BINS>, k_classify<MODE_RANGE1>,
                                                                   k_classify<MODE_RANGE2>, k_classify<MODE_DUMP>};
    hipLaunchKernelGGL(kernels[c.mode], dim3((unsigned)blocks), dim3(CLS), 0, st, c, nA, nB);
    prof_end(pm, st);
    return check_launch("k_classify");
}
}  // namespace

void set_force_exact(int v) { g_force_exact = v; }

void set_distance_stats(long long pairs, long long rechecked, long long exact)
{
    t_pairs = pairs;
    t_rechecked = rechecked;
    t_exact = exact;
}

int last_distance_stats(int64_t *pairs, int64_t *rechecked, int64_t *exact)
{
    if (pairs) *pairs = t_pairs;
    if (rechecked) *rechecked = t_rechecked;
    if (exact) *exact = t_exact;
    return CIL_OK;
}

// Bins / counts for all pairs.  hist_host[M+1] gets the per-bin pair counts.
namespace {

// Bins of every pair from a computed fast pass: classify against the squared
// radii, re-check the listed pairs canonically.  hist_host[m] = #{bin == m}.
template <typename T>
int bins_from_approx(const T *A, long long nA, const T *B, long long nB, long long dim, Approx &ap, DistScratch &s,
                     const double *radii, int M, uint8_t *bins, std::vector<unsigned long long> &hist_host,
                     hipStream_t st)
{
    // pinned staging: [0, 2048) thresholds, [2048, 4096) histogram, [4096, 4112) counters
    char *hs;
    CIL_TRY(host_stage(HS_DIST, 4096 + 64, (void **)&hs));
    double *thr = (double *)hs;
    for (int m = 0; m < M; ++m) thr[m] = radii[m] * radii[m];
    CIL_HIP(hipMemcpyAsync(s.thr, thr, sizeof(double) * M, hipMemcpyHostToDevice, st));
    // the histogram and the two list counters (contiguous) in one clear
    CIL_TRY(fill_zero(s.hist, (char *)(s.nlist + 2) - (char *)s.hist, st));
    ClassifyArgs &c = ap.c;
    c.mode = MODE_BINS;
    c.thr = s.thr;
    c.M = M;
    c.hist = s.hist;
    c.bins = bins;
    c.list = s.list;
    c.nlist = s.nlist;
    c.cap = s.cap;
    CIL_TRY(classify(c, nA, nB, st));
    CanonOut co{};
    co.pairs = s.list;
    co.npairs_dev = s.nlist;
    co.cap = s.cap;
    co.thr = s.thr;
    co.M = M;
    co.hist = s.hist;
    co.bins = bins;
    co.nB = nB;
    co.nexact = s.nexact;
    co.force_exact = g_force_exact;
    const long long guess = std::min(recheck_guess(dim), std::max(s.cap, 1LL));
    CIL_TRY(run_canonical(A, B, dim, co, guess, st));
    unsigned long long *hh = (unsigned long long *)(hs + 2048);
    unsigned long long *cnt = (unsigned long long *)(hs + 4096);   // listed pairs, exact fallbacks
    CIL_HIP(hipMemcpyAsync(hh, s.hist, sizeof(unsigned long long) * (M + 1), hipMemcpyDeviceToHost, st));
    CIL_HIP(hipMemcpyAsync(cnt, s.nlist, 2 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    CIL_TRY(stream_wait(st));
    const unsigned long long nre = cnt[0];
    if ((long long)nre > s.cap) return set_error(CIL_EDEVICE, "re-check list overflow");
    if ((long long)nre > guess) {                       // the rest of a long list
        co.first = guess;
        CIL_TRY(run_canonical(A, B, dim, co, (long long)nre - guess, st));
        CIL_HIP(hipMemcpyAsync(hh, s.hist, sizeof(unsigned long long) * (M + 1), hipMemcpyDeviceToHost, st));
        CIL_HIP(hipMemcpyAsync(cnt, s.nlist, 2 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
        CIL_TRY(stream_wait(st));
    }
    hist_host.assign(hh, hh + M + 1);
    t_pairs = nA * nB;
    t_rechecked = (long long)nre;
    t_exact = (long long)cnt[1];
    return CIL_OK;
}

// Canonical extremes from a computed fast pass: pass 1 bounds them by
// min(D~ + eps) and max(D~ - eps); pass 2 lists every pair whose interval
// reaches those bounds; the listed pairs are recomputed canonically and the
// extremes taken over them.
template <typename T>
int range_from_approx(const T *A, long long nA, const T *B, long long nB, long long dim, Approx &ap, DistScratch &s,
                      int excl, double *dmin, double *dmax, hipStream_t st)
{
    const long long guess = std::min(recheck_guess(dim), std::max(s.cap, 1LL));
    // pinned staging: [0, 40) initial counters, [64, 104) counters read back,
    // [4096, ...) candidate distances read back
    char *hs;
    CIL_TRY(host_stage(HS_DIST, 4096 + sizeof(double) * (size_t)guess, (void **)&hs));
    unsigned long long *init = (unsigned long long *)hs;
    // nlist, nexact, min bound (+inf), max bound (0), non-finite flag
    init[0] = 0ull;
    init[1] = 0ull;
    init[2] = (unsigned long long)0x7ff0000000000000ull;
    init[3] = 0ull;
    init[4] = 0ull;
    CIL_HIP(hipMemcpyAsync(s.nlist, init, 5 * sizeof(unsigned long long), hipMemcpyHostToDevice, st));
    ClassifyArgs &c = ap.c;
    c.exclude_diag = excl;
    c.minmax = s.minmax;
    c.flag = s.flag;
    c.list = s.list;
    c.nlist = s.nlist;
    c.cap = s.cap;
    // pass 1 reads every partial once and leaves their sums, so that pass 2
    // and the bins read one value per pair
    if (c.S > 1) CIL_TRY(ws_get(WS_DIST_REDUCED, sizeof(double) * (size_t)std::max(nA * nB, 1LL), (void **)&c.reduced));
    c.mode = MODE_RANGE1;
    CIL_TRY(classify(c, nA, nB, st));
    if (c.reduced) {
        c.P = c.reduced;
        c.S = 1;
        c.reduced = nullptr;
    }
    c.mode = MODE_RANGE2;                 // stream-ordered after the bounds of pass 1
    CIL_TRY(classify(c, nA, nB, st));
    double *cand;
    CIL_TRY(ws_get(WS_DIST_NORMS, sizeof(double) * (size_t)guess, (void **)&cand));
    CanonOut co{};
    co.pairs = s.list;
    co.npairs_dev = s.nlist;
    co.cap = s.cap;
    co.d2 = cand;
    co.nexact = s.nexact;
    co.force_exact = g_force_exact;
    CIL_TRY(run_canonical(A, B, dim, co, guess, st));
    double *hcp = (double *)(hs + 4096);
    unsigned long long *cnt = (unsigned long long *)(hs + 64);
    CIL_HIP(hipMemcpyAsync(hcp, cand, sizeof(double) * guess, hipMemcpyDeviceToHost, st));
    CIL_HIP(hipMemcpyAsync(cnt, s.nlist, 5 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    CIL_TRY(stream_wait(st));
    std::vector<double> hc(hcp, hcp + guess);
    if (cnt[4]) return set_error(CIL_ENONFINITE, "non-finite distances in range computation");
    const long long nc = (long long)cnt[0];
    if (nc > s.cap) return set_error(CIL_EDEVICE, "range candidate overflow");
    if (nc > guess) {                     // the rest of a long candidate list
        CIL_TRY(ws_get(WS_DIST_NORMS, sizeof(double) * (size_t)nc, (void **)&cand));
        co.d2 = cand;
        co.first = guess;
        CIL_TRY(run_canonical(A, B, dim, co, nc - guess, st));
        hc.resize(nc);
        CIL_HIP(hipMemcpyAsync(hc.data() + guess, cand + guess, sizeof(double) * (nc - guess), hipMemcpyDeviceToHost,
                               st));
        CIL_HIP(hipMemcpyAsync(cnt, s.nlist, 5 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
        CIL_TRY(stream_wait(st));
    }
    double lo = INFINITY, hi = 0.0;
    for (long long k = 0; k < nc; ++k) {
        lo = std::min(lo, hc[k]);
        hi = std::max(hi, hc[k]);
    }
    *dmin = lo;
    *dmax = hi;
    t_pairs = nA * nB;
    t_rechecked = nc;
    t_exact = (long long)cnt[1];
    return CIL_OK;
}

}  // namespace

template <typename T>
int pair_bins_impl(const T *A, long long nA, const T *B, long long nB, long long dim, const double *radii, int M,
                   uint8_t *bins, std::vector<unsigned long long> &hist_host, hipStream_t st)
{
    DistScratch s;
    CIL_TRY(scratch(nA * nB, &s));
    Approx ap;
    CIL_TRY(approx_pass(A, nA, B, nB, dim, &ap, st));
    return bins_from_approx(A, nA, B, nB, dim, ap, s, radii, M, bins, hist_host, st);
}

// Range, radii and bins from one fast pass (the partials stay in their
// workspace between the two classifications).
template <typename T>
int adaptive_bins_impl(const T *A, long long nA, const T *B, long long nB, long long dim, int excl, int M, int law,
                       double *dmin, double *dmax, double *radii, uint8_t *bins,
                       std::vector<unsigned long long> &hist_host, hipStream_t st)
{
    DistScratch s;
    CIL_TRY(scratch(nA * nB, &s));
    Approx ap;
    CIL_TRY(approx_pass(A, nA, B, nB, dim, &ap, st));
    CIL_TRY(range_from_approx(A, nA, B, nB, dim, ap, s, excl, dmin, dmax, st));
    ap.c.exclude_diag = 0;                 // bins of every pair
    const long long nrange = t_rechecked, nrange_exact = t_exact;
    CIL_TRY(radii_ladder(*dmin, *dmax, M, law, radii));
    CIL_TRY(bins_from_approx(A, nA, B, nB, dim, ap, s, radii, M, bins, hist_host, st));
    t_rechecked += nrange;
    t_exact += nrange_exact;
    return CIL_OK;
}

// R_0 - m h rounded as two operations, as the host forms it (no contraction).
__device__ __forceinline__ double linear_radius(double R0, int m, double h)
{
#pragma clang fp contract(off)
    return R0 - (double)m * h;
}

// The device range pass's initial counters, staged in pinned host memory
// (HS_DIST, offset 0; the caller's read-back uses the same buffer further
// on): list count, exact fallbacks, classify bounds (+inf, 0), non-finite
// flag, canonical extremes (+inf, 0), thresholds with a pair near them.
int range_init_stage(unsigned long long **out)
{
    char *hs;
    CIL_TRY(host_stage(HS_DIST, 8192, (void **)&hs));
    unsigned long long *init = (unsigned long long *)hs;
    init[0] = 0ull;
    init[1] = 0ull;
    init[2] = (unsigned long long)0x7ff0000000000000ull;
    init[3] = 0ull;
    init[4] = 0ull;
    init[5] = (unsigned long long)0x7ff0000000000000ull;
    init[6] = 0ull;
    init[7] = 0ull;
    *out = init;
    return CIL_OK;
}

// Range and radii on the device from the range pass's counters (cnt: [0]
// candidates, [1] exact fallbacks, [4] non-finite flag, [5], [6] the
// candidates' canonical extremes): the ladder as the host forms it
// (cil_radii), powers by pow_dd; thr[m] = R_m^2.  A bad range leaves every
// threshold 0 and its status in ro.
__global__ void k_range_radii(const unsigned long long *cnt, long long cap, int M, int law, double *thr, RangeOut *ro)
{
    __shared__ double sR0, sb;
    __shared__ DD slogb;
    __shared__ int sst;
    __shared__ DDTables tab;
    {                                    // the series' coefficients, one per thread
        const int k = threadIdx.x;
        if (k < kLogTerms) tab.inv_odd[k] = dd_inv(2 * k + 1);
        else if (k < kLogTerms + kExpTerms) tab.inv_n[k - kLogTerms + 1] = dd_inv(k - kLogTerms + 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double lo = __longlong_as_double((long long)cnt[5]), hi = __longlong_as_double((long long)cnt[6]);
        ro->d2min = lo;
        ro->d2max = hi;
        ro->nrange = (long long)cnt[0];
        ro->nrange_exact = (long long)cnt[1];
        int st = 0;
        if (cnt[4]) st = 2;
        else if ((long long)cnt[0] > cap) st = 3;
        const double R0 = sqrt_dd(hi), RM = sqrt_dd(lo);
        if (st == 0 && !(RM > 0.0 && R0 > RM && isfinite(R0))) st = 1;
        ro->status = st;
        sst = st;
        sR0 = R0;
        DD lb{0.0, 0.0};
        sb = st != 0 ? 0.0 : (law == 0 ? root_dd(R0 / RM, M, tab, &lb) : (R0 - RM) / M);
        slogb = lb;
    }
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
        double r = 0.0;
        if (sst == 0)
            r = law == 0 ? sR0 * pow_dd_from_log(slogb, (double)-(m + 1), tab) : linear_radius(sR0, m + 1, sb);
        ro->radii[m] = r;
        thr[m] = r * r;
    }
}

// Re-check launches over a list whose length stays on the device: for
// d < 4096 one launch of 2048 slots striding over it; for longer vectors a
// first launch of 256 pairs at sixteen waves each (the usual short list at
// the latency of one pair), then a strided launch of 2048 slots of four waves
// for the rest, which leaves at once when there is none (2769 pairs of d = 32768
// in all 145 us, with single-wave slots 295: wavefronts that walk whole rows at one
// pace from k = 0 on crowd the memory channels).
template <typename T>
int canonical_any_length(const T *A, const T *B, long long dim, CanonOut co, long long cap, hipStream_t st)
{
    if (dim < 4096) {
        co.stride = 2048;
        return run_canonical(A, B, dim, co, 2048, st);
    }
    const long long first = std::min(recheck_guess(dim), std::max(cap, 1LL));
    CIL_TRY(run_canonical(A, B, dim, co, first, st));
    if (cap > first) {
        constexpr long long TAIL = 2048;
        co.first = first;
        co.stride = TAIL;
        const ProfMark pm = prof_begin("k_canonical", st);
        hipLaunchKernelGGL((k_canonical<T, 4>), dim3((unsigned)TAIL), dim3(256), 0, st, A, B, dim, co);
        prof_end(pm, st);
        CIL_TRY(check_launch("k_canonical"));
    }
    return CIL_OK;
}

// The range pass without its read-back: candidates listed as in
// range_from_approx, their canonical distances folded into the device's
// extremes, then the radii and thresholds formed on the device.
template <typename T>
int range_radii_device(const T *A, long long nA, const T *B, long long nB, long long dim, Approx &ap,
                       DistScratch &s, int M, int law, hipStream_t st)
{
    unsigned long long *init;
    CIL_TRY(range_init_stage(&init));
    CIL_HIP(hipMemcpyAsync(s.nlist, init, 8 * sizeof(unsigned long long), hipMemcpyHostToDevice, st));
    ClassifyArgs &c = ap.c;
    c.exclude_diag = 0;
    c.minmax = s.minmax;
    c.flag = s.flag;
    c.list = s.list;
    c.nlist = s.nlist;
    c.cap = s.cap;
    if (c.S > 1) CIL_TRY(ws_get(WS_DIST_REDUCED, sizeof(double) * (size_t)std::max(nA * nB, 1LL), (void **)&c.reduced));
    c.mode = MODE_RANGE1;
    CIL_TRY(classify(c, nA, nB, st));
    if (c.reduced) {
        c.P = c.reduced;
        c.S = 1;
        c.reduced = nullptr;
    }
    c.mode = MODE_RANGE2;
    CIL_TRY(classify(c, nA, nB, st));
    CanonOut co{};
    co.pairs = s.list;
    co.npairs_dev = s.nlist;
    co.cap = s.cap;
    co.range_mm = s.cmm;
    co.nexact = s.nexact;
    co.force_exact = g_force_exact;
    CIL_TRY(canonical_any_length(A, B, dim, co, s.cap, st));
    hipLaunchKernelGGL(k_range_radii, dim3(1), dim3(64), 0, st, s.nlist, s.cap, M, law, s.thr, s.ro);
    return check_launch("k_range_radii");
}

// The same without the bins' read-back: the re-check list is finished on the
// device whatever its length (strided launches), and the
// histogram and list counters stay on the device for the caller's one
// read-back at the end of a longer chain (AsyncBins).  The range and its
// read-back, which the radii need, are as in adaptive_bins_impl.
template <typename T>
int adaptive_bins_async(const T *A, long long nA, const T *B, long long nB, long long dim, int M, int law,
                        int device_radii, double *dmin, double *dmax, double *radii, uint8_t *bins, AsyncBins *ab,
                        hipStream_t st)
{
    DistScratch s;
    CIL_TRY(scratch(nA * nB, &s));
    Approx ap;
    CIL_TRY(approx_pass(A, nA, B, nB, dim, &ap, st));
    if (device_radii) {
        CIL_TRY(range_radii_device(A, nA, B, nB, dim, ap, s, M, law, st));
    } else {
        CIL_TRY(range_from_approx(A, nA, B, nB, dim, ap, s, 0, dmin, dmax, st));
        ab->nrange = t_rechecked;
        ab->nrange_exact = t_exact;
        CIL_TRY(radii_ladder(*dmin, *dmax, M, law, radii));
        char *hs;
        CIL_TRY(host_stage(HS_DIST, 4096 + 64, (void **)&hs));
        double *thr = (double *)hs;
        for (int m = 0; m < M; ++m) thr[m] = radii[m] * radii[m];
        CIL_HIP(hipMemcpyAsync(s.thr, thr, sizeof(double) * M, hipMemcpyHostToDevice, st));
    }
    CIL_TRY(fill_zero(s.hist, (char *)(s.nlist + 2) - (char *)s.hist, st));
    ClassifyArgs &c = ap.c;
    c.exclude_diag = 0;
    c.mode = MODE_BINS;
    c.thr = s.thr;
    // With the device's radii, every pair within 2^-44 thr of a threshold is
    // re-checked and its threshold marked: the host's ladder differs from the
    // device's by a few units in the last place at most (where the C
    // library's pow misrounds), so the bins are those of either ladder unless
    // a marked threshold is one where they differ.
    c.thr_slack = device_radii ? 0x1p-44 : 0.0;
    c.M = M;
    c.hist = s.hist;
    c.bins = bins;
    c.list = s.list;
    c.nlist = s.nlist;
    c.cap = s.cap;
    CIL_TRY(classify(c, nA, nB, st));
    CanonOut co{};
    co.pairs = s.list;
    co.npairs_dev = s.nlist;
    co.cap = s.cap;
    co.thr = s.thr;
    co.M = M;
    co.hist = s.hist;
    co.bins = bins;
    co.nB = nB;
    co.nexact = s.nexact;
    co.force_exact = g_force_exact;
    if (device_radii) {
        co.win_rel = 0x1p-44;
        co.win_hits = s.nlist + 7;
    }
    CIL_TRY(canonical_any_length(A, B, dim, co, s.cap, st));
    ab->hist = s.hist;
    ab->nlist = s.nlist;
    ab->cap = s.cap;
    ab->ro = device_radii ? s.ro : nullptr;
    return CIL_OK;
}

template int adaptive_bins_async<double>(const double *, long long, const double *, long long, long long, int, int,
                                         int, double *, double *, double *, uint8_t *, AsyncBins *, hipStream_t);
template int adaptive_bins_async<float>(const float *, long long, const float *, long long, long long, int, int,
                                        int, double *, double *, double *, uint8_t *, AsyncBins *, hipStream_t);

template int adaptive_bins_impl<double>(const double *, long long, const double *, long long, long long, int, int,
                                        int, double *, double *, double *, uint8_t *,
                                        std::vector<unsigned long long> &, hipStream_t);
template int adaptive_bins_impl<float>(const float *, long long, const float *, long long, long long, int, int, int,
                                       double *, double *, double *, uint8_t *, std::vector<unsigned long long> &,
                                       hipStream_t);

template int pair_bins_impl<double>(const double *, long long, const double *, long long, long long, const double *,
                                    int, uint8_t *, std::vector<unsigned long long> &, hipStream_t);
template int pair_bins_impl<float>(const float *, long long, const float *, long long, long long, const double *, int,
                                   uint8_t *, std::vector<unsigned long long> &, hipStream_t);

template <typename T>
int distance_range_impl(const T *A, long long nA, const T *B, long long nB, long long dim, int excl, double *dmin,
                        double *dmax, hipStream_t st)
{
    DistScratch s;
    CIL_TRY(scratch(nA * nB, &s));
    Approx ap;
    CIL_TRY(approx_pass(A, nA, B, nB, dim, &ap, st));
    return range_from_approx(A, nA, B, nB, dim, ap, s, excl, dmin, dmax, st);
}

template int distance_range_impl<double>(const double *, long long, const double *, long long, long long, int,
                                         double *, double *, hipStream_t);
template int distance_range_impl<float>(const float *, long long, const float *, long long, long long, int, double *,
                                        double *, hipStream_t);

// The fast-pass approximation and its bound for every pair (diagnostics).
template <typename T>
int approx_d2_impl(const T *A, long long nA, const T *B, long long nB, long long dim, double *d2, double *eps,
                   hipStream_t st)
{
    Approx ap;
    CIL_TRY(approx_pass(A, nA, B, nB, dim, &ap, st));
    ap.c.mode = MODE_DUMP;
    ap.c.dump_d = d2;
    ap.c.dump_eps = eps;
    CIL_TRY(classify(ap.c, nA, nB, st));
    t_pairs = nA * nB;
    return CIL_OK;
}

template int approx_d2_impl<double>(const double *, long long, const double *, long long, long long, double *,
                                    double *, hipStream_t);
template int approx_d2_impl<float>(const float *, long long, const float *, long long, long long, double *, double *,
                                   hipStream_t);

// Canonical squared distances of every pair within P sets of n_syn patterns
// (S, back to back) and between n_set patterns and each of those sets:
// D[p][n_syn + n_set][n_syn], the set's own rows first; *nexact counts the exact
// sums on the device.  Stream-ordered.
template <typename T>
int grid_distances_impl(const T *S, int P, long long n_syn, const T *data, long long n_set, long long dim, double *D,
                        unsigned long long **nexact, hipStream_t st)
{
    DistScratch s;
    CIL_TRY(scratch(1, &s));
    CIL_TRY(fill_zero(s.nexact, sizeof(unsigned long long), st));
    *nexact = s.nexact;
    return run_canonical_grid(data, n_set, S, n_syn, n_syn * dim, dim, D, P, nullptr, s.nexact, st);
}
template int grid_distances_impl<double>(const double *, int, long long, const double *, long long, long long, double *,
                                         unsigned long long **, hipStream_t);
template int grid_distances_impl<float>(const float *, int, long long, const float *, long long, long long, double *,
                                        unsigned long long **, hipStream_t);

template <typename T>
int canonical_pairs_impl(const T *A, long long nA, const T *B, long long nB, long long dim, const long long *ia,
                         const long long *jb, long long np, double *d2, hipStream_t st)
{
    DistScratch s;
    CIL_TRY(scratch(1, &s));
    // the list counter slot doubles as the bad-index flag here; nexact counts fallbacks
    CIL_TRY(fill_zero(s.nlist, sizeof(unsigned long long) * 3, st));
    CanonOut co{};
    co.ia = ia;
    co.jb = jb;
    co.npairs = np;
    co.nA = nA;
    co.nB = nB;
    co.bad = (int *)s.nlist;
    co.d2 = d2;
    co.nexact = s.nexact;
    co.force_exact = g_force_exact;
    // A list as long as the grid of all pairs mostly is that grid, row by row:
    // the device looks, and one of the two launches leaves at once (with fewer
    // pairs the shared rows gain nothing: 4608 of d = 32768 173 against 153 us).
    // (The grid kernel reads at least one value of a row.)
    if (np == nA * nB && dim > 0 && grid_gains(nA, nB, dim) && !g_force_exact) {
        int *not_grid = (int *)(s.nlist + 2);
        hipLaunchKernelGGL(k_list_is_grid, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, ia, jb, np, nB, not_grid);
        CIL_TRY(check_launch("k_list_is_grid"));
        CIL_TRY(run_canonical_grid(A, nA, B, nB, 0, dim, d2, 0, not_grid, s.nexact, st));
        co.only_if = not_grid;
    }
    CIL_TRY(run_canonical(A, B, dim, co, np, st));
    unsigned long long *flags;
    CIL_TRY(host_stage(HS_DIST, 4096, (void **)&flags));
    CIL_HIP(hipMemcpyAsync(flags, s.nlist, 2 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    CIL_TRY(stream_wait(st));
    t_pairs = np;
    t_rechecked = np;
    t_exact = (long long)flags[1];
    if (flags[0]) return set_error(CIL_EINVAL, "pair index out of range");
    return CIL_OK;
}

template int canonical_pairs_impl<double>(const double *, long long, const double *, long long, long long,
                                          const long long *, const long long *, long long, double *, hipStream_t);
template int canonical_pairs_impl<float>(const float *, long long, const float *, long long, long long,
                                         const long long *, const long long *, long long, double *, hipStream_t);

}  // namespace cil
