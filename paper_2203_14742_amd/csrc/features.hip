// Pattern features beyond the L2 distance (Sec. 3.1 multi-feature CIL, the
// scaled-data experiments of Sec. 5):
//   * min-max scaling of each species of a pattern;
//   * derivative augmentation: a pattern followed by its forward differences
//     along x and y, so that the W^{1,2} norm of a difference is the L2
//     distance of augmented vectors (the split-bf16x3 Gram path serves it);
//   * max-abs distances per segment of a vector (L-infinity of the pattern,
//     of each derivative), their combination by max (W^{1,inf}) or sum (the
//     W^{1,inf} variant with a sum over derivatives), and the binning of such
//     distances under radii.
//
// Values that decide a bin are exact or correctly rounded:
//   * max_k |a_k - b_k| is taken over fl64(|a_k - b_k|); rounding is monotone,
//     so the result is fl64 of the exact maximum;
//   * scaled and augmented values are formed in FP64 with IEEE operations in a
//     fixed order and rounded once to the pattern's type.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "cil_internal.hpp"

#pragma clang fp contract(off)

namespace cil {

namespace {

template <typename T>
__device__ __forceinline__ double to64(T v) { return (double)v; }

// ---------------------------------------------------------- min-max scaling
// One workgroup per (pattern, species): s~ = (s - min) / (max - min), in FP64,
// rounded to T; a constant species (max == min) maps to 0.
template <typename T>
__global__ __launch_bounds__(256) void k_minmax_scale(const T *X, long long nn, T *Y)
{
    __shared__ double rmin[4], rmax[4];
    const long long base = ((long long)blockIdx.y * 2 + blockIdx.x) * nn;
    const T *x = X + base;
    T *y = Y + base;
    double lo = INFINITY, hi = -INFINITY;
    for (long long k = threadIdx.x; k < nn; k += 256) {
        const double v = to64(x[k]);
        lo = fmin(lo, v);
        hi = fmax(hi, v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o, 64));
        hi = fmax(hi, __shfl_xor(hi, o, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        rmin[threadIdx.x >> 6] = lo;
        rmax[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    lo = fmin(fmin(rmin[0], rmin[1]), fmin(rmin[2], rmin[3]));
    hi = fmax(fmax(rmax[0], rmax[1]), fmax(rmax[2], rmax[3]));
    const double span = hi - lo;
    for (long long k = threadIdx.x; k < nn; k += 256) {
        const double v = to64(x[k]);
        y[k] = span > 0.0 ? (T)((v - lo) / span) : (T)0.0;
    }
}

// ------------------------------------------------------------ augmentation
// Pattern p ([2][n][n]) -> [s (2 n^2) | D_x s (2 n (n-1)) | D_y s (2 n (n-1))],
// D_x s[c][i][j] = (s[c][i][j+1] - s[c][i][j]) / h, j < n - 1;
// D_y s[c][i][j] = (s[c][i+1][j] - s[c][i][j]) / h, i < n - 1.
template <typename T>
__global__ __launch_bounds__(256) void k_augment(const T *X, int n, double h, long long daug, T *Y)
{
    const long long p = blockIdx.y;
    const long long nn = (long long)n * n, ne = (long long)n * (n - 1);
    const T *x = X + p * 2 * nn;
    T *y = Y + p * daug;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < daug; e += (long long)gridDim.x * 256) {
        if (e < 2 * nn) {
            y[e] = x[e];
        } else if (e < 2 * nn + 2 * ne) {
            const long long f = e - 2 * nn, c = f / ne, r = f % ne, i = r / (n - 1), j = r % (n - 1);
            const long long a = c * nn + i * n + j;
            y[e] = (T)((to64(x[a + 1]) - to64(x[a])) / h);
        } else {
            const long long f = e - 2 * nn - 2 * ne, c = f / ne, r = f % ne, i = r / n, j = r % n;
            const long long a = c * nn + i * n + j;
            y[e] = (T)((to64(x[a + n]) - to64(x[a])) / h);
        }
    }
}

// ------------------------------------------------------- max-abs distances
// A wavefront takes 4 x 8 pairs, its lanes along k, so that it reads twelve
// values for thirty-two terms; a workgroup of four 16 x 8 pairs and one K range
// [kb, kb + ksplit).  For each segment [e_{s-1}, e_s) the range meets, the
// partial maxima go to out[(i nB + j) nseg + s] by an atomic max on the bit
// patterns (the values are non-negative doubles, whose order is that of their
// bits), so the result is independent of the order of the K ranges; out starts
// at +0.  Bound by FP64 issue (a subtraction and a maximum a term) and by the L2
// behind it: 62 500 pairs of d = 24320 in FP32, three segments, take 161 us (202 by
// 2 x 8 pairs; 210 by 64 x 64 tiles staged in LDS in FP64).
constexpr int MAX_SEG = 8;
struct SegEnds {
    long long end[MAX_SEG];
};
constexpr int PRW = 4, PCW = 8, PNP = PRW * PCW;         // pairs of a wavefront
constexpr int PTI = 4 * PRW;                              // rows of a workgroup

// max(m, |d|), m where d is not a number: the one instruction (fmax would first
// quieten d, which a subtraction has done).
__device__ __forceinline__ double max_abs(double m, double d)
{
    double r;
    asm("v_max_f64 %0, %1, |%2|" : "=v"(r) : "v"(m), "v"(d));
    return r;
}

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_pair_maxabs(const T *A, long long nA, const T *B, long long nB, long long dim,
                                                     SegEnds ends, int nseg, long long ksplit, unsigned long long *out)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned nct = (unsigned)((nB + PCW - 1) / PCW);
    // in scalars, so that the rows' addresses take no lane registers
    const unsigned bi = __builtin_amdgcn_readfirstlane(blockIdx.x / nct), bj = blockIdx.x - bi * nct;
    const long long i0 = (long long)bi * PTI + PRW * wv, j0 = (long long)bj * PCW;
    const long long kb = (long long)blockIdx.y * ksplit, ke = std::min<long long>(dim, kb + ksplit);
    long long sb = 0;
    for (int s = 0; s < nseg; ++s) {
        const long long se = ends.end[s];
        const long long lo = std::max<long long>(kb, sb), hi = std::min<long long>(ke, se);
        sb = se;
        if (lo >= hi) continue;                     // uniform: this range does not meet segment s
        const T *ra[PRW], *rb[PCW];                 // rows past the end repeat the last (not stored)
#pragma unroll
        for (int r = 0; r < PRW; ++r) ra[r] = A + std::min(i0 + r, nA - 1) * dim + lo;
#pragma unroll
        for (int q = 0; q < PCW; ++q) rb[q] = B + std::min(j0 + q, nB - 1) * dim + lo;
        double m[PNP];
#pragma unroll
        for (int e = 0; e < PNP; ++e) m[e] = 0.0;
        const unsigned len = (unsigned)(hi - lo);
        // blocks start at different k and wrap round: at one k all rows, often a
        // multiple of 1 KB apart, would be on one L2 channel
        const unsigned turn = (bj * 5u + bi * 3u) * 7u % ((len + 63) / 64) * 64u;
        for (int lap = 0; lap < 2; ++lap) {
            unsigned k = (lap ? 0u : turn) + lane;
            const unsigned to = lap ? turn : len;
            if (k >= to) continue;
            T a[PRW], b[PCW];                       // read one round ahead
            auto read = [&](unsigned at) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < PRW; ++r) a[r] = at_byte(ra[r], at * (unsigned)sizeof(T));
#pragma unroll
                for (int q = 0; q < PCW; ++q) b[q] = at_byte(rb[q], at * (unsigned)sizeof(T));
            };
            read(k);
            while (true) {
                double av[PRW], bv[PCW];
#pragma unroll
                for (int r = 0; r < PRW; ++r) av[r] = to64(a[r]);
#pragma unroll
                for (int q = 0; q < PCW; ++q) bv[q] = to64(b[q]);
                k += 64;
                const bool more = k < to;
                read(more ? k : k - 64);
#pragma unroll
                for (int r = 0; r < PRW; ++r)
#pragma unroll
                    for (int q = 0; q < PCW; ++q) m[r * PCW + q] = max_abs(m[r * PCW + q], av[r] - bv[q]);
                if (!more) break;
            }
        }
        // at each level a lane hands over half of its pairs and keeps the rest
        int mine = 0;
#pragma unroll
        for (int half = PNP / 2; half >= 1; half >>= 1) {
            const int off = 64 / PNP * half;
            const bool up = (lane & off) != 0;
            mine += up ? half : 0;
#pragma unroll
            for (int e = 0; e < half; ++e) {
                const double x = m[e], y = m[e + half];
                m[e] = max_abs(up ? y : x, __shfl_xor(up ? x : y, off, 64));
            }
        }
#pragma unroll
        for (int off = 32 / PNP; off >= 1; off >>= 1) m[0] = fmax(m[0], __shfl_xor(m[0], off, 64));
        const long long i = i0 + mine / PCW, j = j0 + mine % PCW;
        if ((lane & (64 / PNP - 1)) == 0 && i < nA && j < nB && m[0] > 0.0)
            atomicMax(&out[(i * nB + j) * nseg + s], (unsigned long long)__double_as_longlong(m[0]));
    }
}

// The same by tiles of 64 x 64 pairs staged through LDS in FP64, 32 values of k at
// a time; thread (ty, tx) owns rows ty + 16 i and columns tx + 16 j, i, j < 4.
// Reads each row once per 64 others and ends a segment with one atomic a pair, so
// it wins where rows are FP64 (the reads through L2 bound k_pair_maxabs there) and
// where segments are short (k_pair_maxabs reduces over its lanes at each end).
constexpr int MT = 64, MKC = 32;
template <typename T>
__global__ __launch_bounds__(256) void k_pair_maxabs_tiles(const T *A, long long nA, const T *B, long long nB,
                                                           long long dim, SegEnds ends, int nseg, long long ksplit,
                                                           unsigned long long *out)
{
    __shared__ double sA[MT][MKC + 1];
    __shared__ double sB[MT][MKC + 1];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const unsigned nct = (unsigned)((nB + MT - 1) / MT);
    const long long i0 = (long long)(blockIdx.x / nct) * MT, j0 = (long long)(blockIdx.x % nct) * MT;
    const long long kb = (long long)blockIdx.y * ksplit, ke = std::min<long long>(dim, kb + ksplit);
    long long sb = 0;
    for (int s = 0; s < nseg; ++s) {
        const long long se = ends.end[s];
        const long long lo = std::max<long long>(kb, sb), hi = std::min<long long>(ke, se);
        sb = se;
        if (lo >= hi) continue;                     // uniform: this range does not meet segment s
        double m[4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) m[a][b] = 0.0;
        for (long long k0 = lo; k0 < hi; k0 += MKC) {
            __syncthreads();
            for (int e = tid; e < MT * MKC; e += 256) {
                const int r = e / MKC, kk = e % MKC;
                const long long k = k0 + kk, ia = i0 + r, jb = j0 + r;
                // positions past the range repeat its first element: |a - b|
                // there is one of the range's own terms, so the max is unchanged
                const long long kc = k < hi ? k : k0;
                sA[r][kk] = ia < nA ? to64(A[ia * dim + kc]) : 0.0;
                sB[r][kk] = jb < nB ? to64(B[jb * dim + kc]) : 0.0;
            }
            __syncthreads();
#pragma unroll 8
            for (int kk = 0; kk < MKC; ++kk) {
                double av[4], bv[4];
#pragma unroll
                for (int a = 0; a < 4; ++a) av[a] = sA[ty + 16 * a][kk];
#pragma unroll
                for (int b = 0; b < 4; ++b) bv[b] = sB[tx + 16 * b][kk];
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int b = 0; b < 4; ++b) m[a][b] = fmax(m[a][b], fabs(av[a] - bv[b]));
            }
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const long long i = i0 + ty + 16 * a, j = j0 + tx + 16 * b;
                if (i < nA && j < nB && m[a][b] > 0.0)
                    atomicMax(&out[(i * nB + j) * nseg + s], (unsigned long long)__double_as_longlong(m[a][b]));
            }
    }
}

// out[p] over D[p][0..nseg-1]: mode 0 max, 1 left-to-right sum, 2 left-to-right
// sum of the (correctly rounded) square roots
__global__ void k_combine(const double *D, long long n, int nseg, int mode, double *out)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const double *d = D + p * nseg;
    double v = mode == 2 ? sqrt(d[0]) : d[0];
    for (int s = 1; s < nseg; ++s) v = mode == 0 ? fmax(v, d[s]) : v + (mode == 2 ? sqrt(d[s]) : d[s]);
    out[p] = v;
}

// min and max of V (as ordered bit patterns of non-negative doubles, the minimum
// as the largest complement, so both start at 0).
__global__ __launch_bounds__(256) void k_value_range(const double *V, long long n, unsigned long long *mm)
{
    __shared__ unsigned long long rlo[4], rhi[4];
    unsigned long long lo = ~0ull, hi = 0ull;
    for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) {
        const unsigned long long b = __double_as_longlong(V[p]);
        lo = b < lo ? b : lo;
        hi = b > hi ? b : hi;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long l2 = __shfl_xor(lo, o, 64), h2 = __shfl_xor(hi, o, 64);
        lo = l2 < lo ? l2 : lo;
        hi = h2 > hi ? h2 : hi;
    }
    if ((threadIdx.x & 63) == 0) {
        rlo[threadIdx.x >> 6] = lo;
        rhi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) {
            lo = rlo[w] < lo ? rlo[w] : lo;
            hi = rhi[w] > hi ? rhi[w] : hi;
        }
        atomicMax(&mm[0], ~lo);
        atomicMax(&mm[1], hi);
    }
}

// bins[p] = #{m : V[p] < radii[m]} (radii decreasing), hist[b] += 1
constexpr int VMAX_M = 255;
__global__ __launch_bounds__(256) void k_bin_values(const double *V, long long n, const double *radii, int M,
                                                    uint8_t *bins, unsigned long long *hist)
{
    __shared__ double r[VMAX_M];
    __shared__ unsigned int h[VMAX_M + 1];
    for (int m = threadIdx.x; m < M; m += 256) r[m] = radii[m];
    for (int m = threadIdx.x; m <= M; m += 256) h[m] = 0;
    __syncthreads();
    for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) {
        const double v = V[p];
        int c = 0;
        while (c < M && v < r[c]) ++c;
        if (bins) bins[p] = (uint8_t)c;
        atomicAdd(&h[c], 1u);
    }
    __syncthreads();
    for (int m = threadIdx.x; m <= M; m += 256)
        if (h[m]) atomicAdd(&hist[m], (unsigned long long)h[m]);
}

unsigned grid_for(long long n, long long cap)
{
    return (unsigned)std::max<long long>(1, std::min<long long>(cap, (n + 255) / 256));
}

// Workgroups of the passes over n values.  Their closing atomics all go to a few
// addresses (22 ns a workgroup for the range, 25 for ten bins), so few values take
// few workgroups; many need more in flight.  us at 512 / 1024 / 2048 / 4096:
//   range         1e6 32 / 44 / 67 / 109, 1e7 52 / 55 / 76 / 118, 3e7 94 / 79 / 95 / 130, 1e8 368 / 234 / 188 / 216
//   bins, M = 10  1e6 42 / 45 / 56 / 125, 4e6 67 / 59 / 63 / 142, 1e7 117 / 87 / 82 / 162, 1e8 1007 / 606 / 503 / 480
//   bins, M = 255 3e5 94 / 73 / 77 / 76, 1e6 202 / 161 / 145 / 154, 2e6 358 / 260 / 233 / 225, 1e8 16435 / .. / 9427
unsigned range_grid(long long n) { return grid_for(n, n <= 10000000 ? 512 : n <= 60000000 ? 1024 : 2048); }
unsigned bins_grid(long long n, int M)
{
    const double q = (double)n * (M + 10);               // the threshold search grows with M
    return grid_for(n, q < 4e7 ? 512 : q < 1.3e8 ? 1024 : q < 5e8 ? 2048 : 4096);
}

// The max-abs kernel's workgroups and its split of k: about 1024 tiles staged in
// LDS, or 2048 workgroups of wavefronts in parts of at least 256.
struct MaxabsGrid {
    bool lds;
    long long tiles, splits, ks;
};
MaxabsGrid maxabs_grid(bool lds, long long nA, long long nB, long long dim)
{
    const long long ti = lds ? MT : PTI, tj = lds ? MT : PCW, part = lds ? MKC : 256, full = lds ? 1024 : 2048;
    const long long tiles = ((nA + ti - 1) / ti) * ((nB + tj - 1) / tj), chunks = (dim + part - 1) / part;
    const long long splits = std::max<long long>({1, std::min<long long>(chunks, (full + tiles - 1) / tiles),
                                                  (dim + (1ll << 28) - 1) >> 28});
    const long long ks = (chunks + splits - 1) / splits * part;
    return MaxabsGrid{lds, tiles, (dim + ks - 1) / ks, ks};
}
// The faster of the two, by a fit to 890 sizes (1 x 1000 to 4000 x 4000 pairs, d = 8
// .. 24320, 1, 3 and 8 segments): a call's overhead, the terms of its padded
// pairs, and per segment met the reduction over the lanes or the atomics (whose
// lines the segments of a pair share).  us, wavefronts / tiles: FP64 250^2 of d =
// 8192 122 / 102, 1000^2 of 2048 381 / 244, of 24320 4866 / 2526; FP32 250^2 of 24320
// 174 / 201, 1000^2 of 200 73 / 63, 2048^2 of 20 148 / 60, of 8192 2677 / 3238; three
// segments 1000^2 of 200 115 / 127, 2048^2 of 20 343 / 223.
MaxabsGrid choose_maxabs(long long nA, long long nB, long long dim, int nseg, cil_precision prec)
{
    const MaxabsGrid w = maxabs_grid(false, nA, nB, dim), t = maxabs_grid(true, nA, nB, dim);
    const double np = (double)nA * nB, d = (double)dim;
    auto met = [&](const MaxabsGrid &g) { return (double)(nseg > 1 ? nseg + g.splits - 1 : g.splits); };
    double tw = 31.0 + (double)w.tiles * PTI * PCW * (2.2e-5 * met(w) + (prec == CIL_FP32 ? 8.1e-8 : 1.6e-7) * d);
    double tt = 40.0 + (double)t.tiles * MT * MT * 9.4e-8 * (d + 16.0 * nseg);
    if (nseg > 1) {
        tw += np * 7.5e-6 * met(w);
        tt += np * 3.8e-6 * nseg * met(t);
    }
    return tt < tw ? t : w;
}

}  // namespace

int minmax_scale_impl(const void *X, long long count, int n, cil_precision prec, void *Y, hipStream_t st)
{
    if (count == 0) return CIL_OK;
    const long long nn = (long long)n * n;
    dim3 grid(2, (unsigned)count);
    if (prec == CIL_FP32)
        hipLaunchKernelGGL(k_minmax_scale<float>, grid, dim3(256), 0, st, (const float *)X, nn, (float *)Y);
    else
        hipLaunchKernelGGL(k_minmax_scale<double>, grid, dim3(256), 0, st, (const double *)X, nn, (double *)Y);
    return check_launch("k_minmax_scale");
}

int augment_impl(const void *X, long long count, int n, double L, cil_precision prec, void *Y, hipStream_t st)
{
    if (count == 0) return CIL_OK;
    const long long daug = 2ll * n * n + 4ll * n * (n - 1);
    const double h = L / (double)(n - 1);
    dim3 grid((unsigned)std::min<long long>(64, (daug + 255) / 256), (unsigned)count);
    if (prec == CIL_FP32)
        hipLaunchKernelGGL(k_augment<float>, grid, dim3(256), 0, st, (const float *)X, n, h, daug, (float *)Y);
    else
        hipLaunchKernelGGL(k_augment<double>, grid, dim3(256), 0, st, (const double *)X, n, h, daug, (double *)Y);
    return check_launch("k_augment");
}

int pair_maxabs_impl(const void *A, long long nA, const void *B, long long nB, long long dim, cil_precision prec,
                     const int64_t *seg_end, int nseg, double *D, hipStream_t st)
{
    if (nseg < 1 || nseg > MAX_SEG) return set_error(CIL_EINVAL, "nseg must be in [1, %d]", MAX_SEG);
    long long prev = 0;
    for (int s = 0; s < nseg; ++s) {
        if (seg_end[s] < prev || seg_end[s] > dim) return set_error(CIL_EINVAL, "segment ends must rise to <= dim");
        prev = seg_end[s];
    }
    if (nA * nB == 0) return CIL_OK;
    CIL_TRY(fill_zero(D, sizeof(double) * (size_t)(nA * nB * nseg), st));
    if (dim == 0) return CIL_OK;
    SegEnds ends{};
    for (int s = 0; s < nseg; ++s) ends.end[s] = seg_end[s];
    unsigned long long *out = (unsigned long long *)D;
    const MaxabsGrid g = choose_maxabs(nA, nB, dim, nseg, prec);
    const char *name = g.lds ? "k_pair_maxabs_tiles" : "k_pair_maxabs";
    const dim3 grid((unsigned)g.tiles, (unsigned)g.splits);
    const ProfMark pm = prof_begin(name, st);
    if (prec == CIL_FP32)
        hipLaunchKernelGGL(g.lds ? k_pair_maxabs_tiles<float> : k_pair_maxabs<float>, grid, dim3(256), 0, st,
                           (const float *)A, nA, (const float *)B, nB, dim, ends, nseg, g.ks, out);
    else
        hipLaunchKernelGGL(g.lds ? k_pair_maxabs_tiles<double> : k_pair_maxabs<double>, grid, dim3(256), 0, st,
                           (const double *)A, nA, (const double *)B, nB, dim, ends, nseg, g.ks, out);
    prof_end(pm, st);
    return check_launch(name);
}

int combine_segments_impl(const double *D, long long n, int nseg, int mode, double *out, hipStream_t st)
{
    if (n == 0) return CIL_OK;
    hipLaunchKernelGGL(k_combine, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, D, n, nseg, mode, out);
    return check_launch("k_combine");
}

int value_range_impl(const double *V, long long n, double *vmin, double *vmax, hipStream_t st)
{
    void *p;
    CIL_TRY(ws_get(WS_FEAT_MISC, 2 * sizeof(unsigned long long), &p));
    unsigned long long *mm = (unsigned long long *)p, *h;
    CIL_TRY(host_stage(HS_FEAT, 4096, (void **)&h));
    CIL_TRY(fill_zero(mm, 2 * sizeof(unsigned long long), st));
    hipLaunchKernelGGL(k_value_range, dim3(range_grid(n)), dim3(256), 0, st, V, n, mm);
    CIL_TRY(check_launch("k_value_range"));
    CIL_HIP(hipMemcpyAsync(h, mm, 2 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    CIL_TRY(stream_wait(st));
    const unsigned long long lo = ~h[0], hi = h[1];
    std::memcpy(vmin, &lo, 8);
    std::memcpy(vmax, &hi, 8);
    return CIL_OK;
}

int bin_values_impl(const double *V, long long n, const double *radii, int M, uint8_t *bins, int64_t *counts,
                    hipStream_t st)
{
    if (M < 1 || M > VMAX_M) return set_error(CIL_EINVAL, "M must be in [1, %d]", VMAX_M);
    void *p;
    CIL_TRY(ws_get(WS_FEAT_MISC, sizeof(unsigned long long) * (M + 1) + sizeof(double) * M, &p));
    unsigned long long *hist = (unsigned long long *)p;
    double *dr = (double *)(hist + M + 1);
    CIL_TRY(fill_zero(hist, sizeof(unsigned long long) * (M + 1), st));
    char *h;
    CIL_TRY(host_stage(HS_FEAT, 4096, (void **)&h));
    std::memcpy(h, radii, sizeof(double) * M);
    CIL_HIP(hipMemcpyAsync(dr, h, sizeof(double) * M, hipMemcpyHostToDevice, st));
    if (n > 0) {
        hipLaunchKernelGGL(k_bin_values, dim3(bins_grid(n, M)), dim3(256), 0, st, V, n, dr, M, bins, hist);
        CIL_TRY(check_launch("k_bin_values"));
    }
    unsigned long long *hh = (unsigned long long *)(h + sizeof(double) * VMAX_M);
    CIL_HIP(hipMemcpyAsync(hh, hist, sizeof(unsigned long long) * (M + 1), hipMemcpyDeviceToHost, st));
    CIL_TRY(stream_wait(st));
    unsigned long long tail = 0;
    for (int m = M; m >= 1; --m) {
        tail += hh[m];
        counts[m - 1] = (int64_t)tail;
    }
    return CIL_OK;
}

}  // namespace cil
