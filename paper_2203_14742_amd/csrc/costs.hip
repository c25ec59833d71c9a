// The synthetic-likelihood cost of a batch of proposals (Alg. 3bst, eq.
// cil:CF_synth) from their synthetic patterns, all proposals in each launch.
//
// Per proposal the pairs are few (64 synthetic patterns, 8 data patterns: 2528)
// and the vectors long, so every distance is formed canonically (k_canonical_grid)
// and the range, bins and resamples read them directly: nothing is approximated,
// listed or re-checked.  The host forms the radii from the ranges, as for the
// other calls, and waits once for those and once for the costs.  20 proposals of
// 64 stationary patterns of 128^2 take 591 us (of noise, whose sums end on a rounding
// boundary more often and are then formed twice, 688); one proposal after the
// other through the pair-statistic calls, with four waits and two dozen launches
// each, take 6280.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "cil_internal.hpp"

namespace cil {

template <typename T>
int grid_distances_impl(const T *, int, long long, const T *, long long, long long, double *, unsigned long long **,
                        hipStream_t);
int loglik_impl(const double *, int, int, int, const double *, double *, double *, int *, int *, hipStream_t);
void set_distance_stats(long long, long long, long long);

namespace {

// Extremes of the distances between distinct patterns of each set, and whether
// one is not finite; one workgroup per proposal.
struct CostRange {
    double lo, hi;
    int bad, pad;
};
__global__ __launch_bounds__(256) void k_cost_range(const double *D, long long n_syn, long long stride, CostRange *out)
{
    __shared__ double slo[4], shi[4];
    __shared__ int sbad[4];
    const double *d = D + blockIdx.x * stride;
    double lo = INFINITY, hi = 0.0;
    int bad = 0;
    for (long long e = threadIdx.x; e < n_syn * n_syn; e += 256) {
        const long long i = e / n_syn, j = e % n_syn;
        if (j <= i) continue;
        const double v = d[e];
        bad |= !isfinite(v);
        lo = fmin(lo, v);
        hi = fmax(hi, v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o, 64));
        hi = fmax(hi, __shfl_xor(hi, o, 64));
        bad |= __shfl_xor(bad, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        slo[threadIdx.x >> 6] = lo;
        shi[threadIdx.x >> 6] = hi;
        sbad[threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) {
            lo = fmin(lo, slo[w]);
            hi = fmax(hi, shi[w]);
            bad |= sbad[w];
        }
        out[blockIdx.x] = CostRange{lo, hi, bad, 0};
    }
}

// bins[e] = #{m : D[e] < thr[p][m]} (thresholds falling)
__global__ __launch_bounds__(256) void k_cost_bins(const double *D, long long stride, const double *thr, int M,
                                                   uint8_t *bins)
{
    __shared__ double t[64];
    const long long p = blockIdx.y;
    if (threadIdx.x < M) t[threadIdx.x] = thr[p * M + threadIdx.x];
    __syncthreads();
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= stride) return;
    const double d = D[p * stride + e];
    int c = 0;
    for (int m = 0; m < M; ++m) c += d < t[m];
    bins[p * stride + e] = (uint8_t)c;
}

// One wavefront per resample vector, and one more per proposal for the observed
// vector (all data rows, the subset's columns).  Lane m keeps the count of
// threshold m (M <= 64): each round of 64 pairs adds the set bits of one ballot
// a threshold.
__global__ __launch_bounds__(256) void k_cost_vectors(const uint8_t *bins, long long n_syn, long long n_set, int M,
                                                      const int *idx1, int k1, const int *idx2, int k2,
                                                      const int *subset, int ks, int n_boot, double *Y, double *yobs,
                                                      int *bad)
{
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long p = blockIdx.y;
    if (r > n_boot) return;
    const bool obs = r == n_boot;
    const uint8_t *b = bins + p * (n_syn + n_set) * n_syn;
    const int rows = obs ? (int)n_set : k1, cols = obs ? ks : k2;
    const int *ri = idx1 + (long long)r * k1, *ci = obs ? subset : idx2 + (long long)r * k2;
    const int pairs = rows * cols;
    unsigned cnt = 0;
    for (int e0 = 0; e0 < pairs; e0 += 64) {
        const int e = e0 + lane;
        int v = 0;
        if (e < pairs) {
            const int a = e / cols, c = e - a * cols;
            const long long i = obs ? n_syn + a : (long long)ri[a], j = ci[c];
            if ((!obs && (i < 0 || i >= n_syn)) || j < 0 || j >= n_syn) atomicOr(bad, 1);
            else v = b[i * n_syn + j];
        }
        for (int m = 0; m < M; ++m) {
            const unsigned c = __popcll(__ballot(v > m));
            cnt += lane == m ? c : 0u;
        }
    }
    if (lane < M) {
        const double y = (double)cnt / ((double)rows * (double)cols);
        if (obs) yobs[p * M + lane] = y;
        else Y[(p * n_boot + r) * M + lane] = y;
    }
}

int costs_of_group(const void *S, int P, long long n_syn, const void *data, long long n_set, long long dim,
                   cil_precision prec, int M, int law, const int *idx1, int k1, const int *idx2, int k2,
                   const int *subset, int ks, int n_boot, double *f, double *loglik, int *status, long long *exact, hipStream_t st)
{
    const long long stride = (n_syn + n_set) * n_syn;
    // device: distances, thresholds, vectors, likelihood outputs, flag, bins
    size_t off = 0;
    auto carve = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t oD = carve(sizeof(double) * P * stride), oT = carve(sizeof(double) * P * M),
                 oY = carve(sizeof(double) * P * n_boot * M), oO = carve(sizeof(double) * P * M),
                 oF = carve(sizeof(double) * 2 * P + sizeof(int) * (2 * P + 2)), oB = carve((size_t)P * stride),
                 oG = carve(sizeof(CostRange) * P);
    char *w;
    CIL_TRY(ws_get(WS_COSTS, off, (void **)&w));
    double *D = (double *)(w + oD), *thr = (double *)(w + oT), *Y = (double *)(w + oY), *yobs = (double *)(w + oO);
    double *df = (double *)(w + oF), *dl = df + P;
    int *dst = (int *)(dl + P), *dme = dst + P, *dbad = dme + P;
    uint8_t *bins = (uint8_t *)(w + oB);
    CostRange *drg = (CostRange *)(w + oG);
    // pinned: ranges, thresholds, results
    const size_t hT = sizeof(CostRange) * P, hR = hT + sizeof(double) * P * M;
    const size_t rbytes = sizeof(double) * 2 * P + sizeof(int) * (2 * P + 2);
    char *h;
    CIL_TRY(host_stage(HS_COSTS, hR + rbytes + sizeof(unsigned long long), (void **)&h));
    CostRange *rg = (CostRange *)h;
    double *hthr = (double *)(h + hT);
    unsigned long long *dexact, *hexact = (unsigned long long *)(h + hR + rbytes);
    if (prec == CIL_FP64)
        CIL_TRY(grid_distances_impl((const double *)S, P, n_syn, (const double *)data, n_set, dim, D, &dexact, st));
    else
        CIL_TRY(grid_distances_impl((const float *)S, P, n_syn, (const float *)data, n_set, dim, D, &dexact, st));
    hipLaunchKernelGGL(k_cost_range, dim3(P), dim3(256), 0, st, D, n_syn, stride, drg);
    CIL_TRY(check_launch("k_cost_range"));
    CIL_HIP(hipMemcpyAsync(rg, drg, sizeof(CostRange) * P, hipMemcpyDeviceToHost, st));
    CIL_TRY(fill_zero(dst, (sizeof(int) * (2 * P + 2) + 7) / 8 * 8, st));
    CIL_TRY(stream_wait(st));
    std::vector<char> degenerate(P, 0);
    std::vector<double> radii(M);
    for (int p = 0; p < P; ++p) {
        if (rg[p].bad) return set_error(CIL_ENONFINITE, "non-finite distances in range computation");
        degenerate[p] = radii_ladder(rg[p].lo, rg[p].hi, M, law, radii.data()) != CIL_OK;
        for (int m = 0; m < M; ++m) hthr[(size_t)p * M + m] = degenerate[p] ? 0.0 : radii[m] * radii[m];
    }
    clear_error();
    CIL_HIP(hipMemcpyAsync(thr, hthr, sizeof(double) * P * M, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_cost_bins, dim3((unsigned)((stride + 255) / 256), P), dim3(256), 0, st, D, stride, thr, M, bins);
    CIL_TRY(check_launch("k_cost_bins"));
    hipLaunchKernelGGL(k_cost_vectors, dim3((unsigned)((n_boot + 4) / 4), P), dim3(256), 0, st, bins, n_syn, n_set, M, idx1,
                       k1, idx2, k2, subset, ks, n_boot, Y, yobs, dbad);
    CIL_TRY(check_launch("k_cost_vectors"));
    CIL_TRY(loglik_impl(Y, P, n_boot, M, yobs, df, dl, dme, dst, st));
    CIL_HIP(hipMemcpyAsync(h + hR, df, rbytes, hipMemcpyDeviceToHost, st));
    CIL_HIP(hipMemcpyAsync(hexact, dexact, sizeof(*hexact), hipMemcpyDeviceToHost, st));
    CIL_TRY(stream_wait(st));
    const double *hf = (const double *)(h + hR), *hl = hf + P;
    const int *hs = (const int *)(hl + P), *hbad = hs + 2 * P;
    if (*hbad) return set_error(CIL_EINVAL, "resample index out of range");
    for (int p = 0; p < P; ++p) {
        f[p] = degenerate[p] ? NAN : hf[p];
        loglik[p] = degenerate[p] ? NAN : hl[p];
        status[p] = degenerate[p] ? CIL_EINVAL : hs[p];
    }
    *exact += (long long)*hexact;
    return CIL_OK;
}

}  // namespace

int synthetic_costs_impl(const void *S, int P, long long n_syn, const void *data, long long n_set, long long dim,
                         cil_precision prec, int M, int law, const int *idx1, int k1, const int *idx2, int k2,
                         const int *subset, int ks, int n_boot, double *f, double *loglik, int *status, hipStream_t st)
{
    // as many proposals at a time as 256 MB hold the distances, bins and vectors of
    const long long stride = (n_syn + n_set) * n_syn, each = 9 * stride + 8ll * n_boot * M;
    const int group = (int)std::max(1ll, std::min((long long)P, (1ll << 28) / each));
    long long exact = 0;
    for (int p = 0; p < P; p += group)
        CIL_TRY(costs_of_group((const char *)S + p * n_syn * dim * (prec == CIL_FP64 ? 8 : 4), std::min(group, P - p), n_syn,
                               data, n_set, dim, prec, M, law, idx1, k1, idx2, k2, subset, ks, n_boot, f + p, loglik + p,
                               status + p, &exact, st));
    set_distance_stats(P * stride, P * stride, exact);
    return CIL_OK;
}

}  // namespace cil
