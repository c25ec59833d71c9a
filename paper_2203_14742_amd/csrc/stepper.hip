// Batched IMEX-Euler reaction-diffusion stepper (App. B.1.1 method-of-lines
// system of the Sec. 4.1 models) on gfx950.
//
// One step of one solve, both species s in {v, w}:
//   r_s   = u_s + dt F_s(u_v, u_w)                   (explicit, old values)
//   u_s'  = (I - dt nu_s Lap_h)^{-1} r_s              (implicit diffusion)
// Lap_h is the five-point Laplacian with ghost-copy Neumann boundaries; its
// eigenvectors are the cosine modes cos(pi k (i+1/2)/n) with eigenvalues
// -(4/h^2)(sin^2(pi k/2n) + sin^2(pi l/2n)), so the solve is: 2D DCT-II,
// divide by 1 + dt nu_s Lambda_kl, inverse 2D DCT.
//
// Three back-ends:
//   plain  one kernel per stage (reaction, row DCT, column DCT + divide,
//          column inverse, row inverse + residual), dense cosine matrices,
//          state streamed through HBM, host-driven step loop; any n >= 2.
//   fused  one persistent workgroup per solve, the whole n x n x 2 state
//          resident in LDS from the first step to the last; every line
//          transformed in registers, on the matrix cores (dct_mfma.hpp; any n
//          up to 128 in FP32, 96 in FP64), by one lane (dct_reg.hpp) or by a
//          quad of lanes (dct_quad.hpp; n in {32, 64, 128} in FP32, {32, 64}
//          in FP64); the workgroup evaluates its own stop rule and retires.
//   tiled  (stepper_split.hip) the matrix-core transforms with a wavefront per
//          eight lines and a launch per pass over all solves, the field in
//          memory, the plain back-end's step loop; n in 65 .. 128.
// All evaluate the stationarity residual max |u^s - u^{s-1}| / dt in FP64
// every check_every steps (and at max_steps), per solve.  FP32 solves whose
// residual falls below the FP32 floor continue in FP64 (phase 2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <tuple>
#include <vector>

#include "cil_internal.hpp"
#include "dct_reg.hpp"
#include "stepper_common.hpp"

namespace cil {

__global__ void k_clear_results(const int *list, int nlist, StepResults R)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < nlist) {
        int b = list[t];
        R.resid[b] = 0ull;
        R.maxabs[b] = 0ull;
        R.bad[b] = 0;
    }
}

// ======================================================================
// Plain back-end.  Work buffers are [slot][2][n][n] in T.  Tables per n:
// C[k][j] = cos(pi k (2j+1)/2n), Ct = C^T, Cw[k][j] = w_k C[k][j] with
// w_0 = 1/n, w_k = 2/n (so Cw^T inverts C), lam[k] = 4 sin^2(pi k/2n).

template <typename T>
__global__ void k_plain_reaction(const DevSolve *S, const int *list, const T *state, T *R,
                                 int n, int model, double dt)
{
    const int slot = blockIdx.y;
    const DevSolve s = S[list[slot]];
    const int N2 = n * n;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N2) return;
    const T *u = state + s.off;
    T *r = R + (size_t)slot * 2 * N2;
    T p[4] = {T(s.p[0]), T(s.p[1]), T(s.p[2]), T(s.p[3])};
    const T v = u[q], w = u[N2 + q];
    dispatch_model(model, [&](auto MD) {
        T f, g;
        kinetics<MD>(p, v, w, f, g);
        r[q] = v + T(dt) * f;
        r[N2 + q] = w + T(dt) * g;
    });
}

// Second-order IMEX reaction stage (semi-implicit BDF2): with the history
// uh = u^{s-2}, fh = F(u^{s-2}) (same layout as the state),
//   r = (4 u^{s-1} - u^{s-2}) / 3 + (2 dt / 3) (2 F(u^{s-1}) - F(u^{s-2})),
// followed by the diffusion solve with 2 dt / 3 in place of dt.  The first
// step of a call is the IMEX-Euler stage (no history yet).  Either way the
// history moves on to u^{s-1}, F(u^{s-1}).
template <typename T>
__global__ void k_plain_reaction_sbdf2(const DevSolve *S, const int *list, const T *state, T *R, T *uh, T *fh,
                                       int n, int model, double dt, int first)
{
    const int slot = blockIdx.y;
    const DevSolve s = S[list[slot]];
    const int N2 = n * n;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N2) return;
    const T *u = state + s.off;
    T *up = uh + s.off, *fp = fh + s.off;
    T *r = R + (size_t)slot * 2 * N2;
    T p[4] = {T(s.p[0]), T(s.p[1]), T(s.p[2]), T(s.p[3])};
    const T v = u[q], w = u[N2 + q];
    dispatch_model(model, [&](auto MD) {
        T f, g;
        kinetics<MD>(p, v, w, f, g);
        if (first) {
            r[q] = v + T(dt) * f;
            r[N2 + q] = w + T(dt) * g;
        } else {
            const T c = T(2.0 * dt / 3.0), third = T(1.0 / 3.0);
            r[q] = (T(4) * v - up[q]) * third + c * (T(2) * f - fp[q]);
            r[N2 + q] = (T(4) * w - up[N2 + q]) * third + c * (T(2) * g - fp[N2 + q]);
        }
        up[q] = v;
        up[N2 + q] = w;
        fp[q] = f;
        fp[N2 + q] = g;
    });
}

// out[i][l] = sum_j in[i][j] C[l][j]   (row forward)
template <typename T>
__global__ void k_plain_rows_fwd(const int *list, const T *in, T *out, const T *Ct, int n)
{
    const int slot = blockIdx.y;
    const int N2 = n * n;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 2 * N2) return;
    (void)list;
    const int sp = e / N2, i = (e / n) % n, l = e % n;
    const T *x = in + (size_t)slot * 2 * N2 + (size_t)sp * N2 + (size_t)i * n;
    T acc = T(0);
    #pragma unroll 8
    for (int j = 0; j < n; ++j) acc += x[j] * Ct[j * n + l];
    out[(size_t)slot * 2 * N2 + e] = acc;
}

// out[k][l] = S_kl * sum_i C[k][i] in[i][l],  S_kl = 1/(1 + dt nu (lam_k+lam_l)/h^2)
template <typename T>
__global__ void k_plain_cols_fwd_div(const DevSolve *S, const int *list, const T *in, T *out,
                                     const T *C, const double *lam, int n, double dt)
{
    const int slot = blockIdx.y;
    const DevSolve s = S[list[slot]];
    const int N2 = n * n;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 2 * N2) return;
    const int sp = e / N2, k = (e / n) % n, l = e % n;
    const T *x = in + (size_t)slot * 2 * N2 + (size_t)sp * N2;
    T acc = T(0);
    #pragma unroll 8
    for (int i = 0; i < n; ++i) acc += C[k * n + i] * x[i * n + l];
    const double nu = sp ? s.nu[1] : s.nu[0];     // a select: an indexed read would place s in memory
    const double fac = 1.0 / (1.0 + dt * nu * (lam[k] + lam[l]) * s.inv_h2);
    out[(size_t)slot * 2 * N2 + e] = acc * T(fac);
}

// out[i][l] = sum_k Cw[k][i] in[k][l]   (column inverse)
template <typename T>
__global__ void k_plain_cols_inv(const int *list, const T *in, T *out, const T *Cw, int n)
{
    const int slot = blockIdx.y;
    (void)list;
    const int N2 = n * n;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 2 * N2) return;
    const int sp = e / N2, i = (e / n) % n, l = e % n;
    const T *x = in + (size_t)slot * 2 * N2 + (size_t)sp * N2;
    T acc = T(0);
    #pragma unroll 8
    for (int k = 0; k < n; ++k) acc += Cw[k * n + i] * x[k * n + l];
    out[(size_t)slot * 2 * N2 + e] = acc;
}

// u'[i][j] = sum_l in[i][l] Cw[l][j]   (row inverse), written to the state;
// at an evaluation step also the residual against the old state.
template <typename T>
__global__ void k_plain_rows_inv(const DevSolve *S, const int *list, const T *in, T *state,
                                 const T *Cw, int n, int check, StepResults R)
{
    const int slot = blockIdx.y;
    const int b = list[slot];
    const DevSolve s = S[b];
    const int N2 = n * n;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    double d = 0.0, a = 0.0;
    int bad = 0;
    if (e < 2 * N2) {
        const int sp = e / N2, i = (e / n) % n, j = e % n;
        const T *x = in + (size_t)slot * 2 * N2 + (size_t)sp * N2 + (size_t)i * n;
        T acc = T(0);
        #pragma unroll 8
        for (int l = 0; l < n; ++l) acc += x[l] * Cw[l * n + j];
        T *u = state + s.off;
        if (check) {
            const double old = (double)u[e];
            d = fabs((double)acc - old);
            a = fabs((double)acc);
            bad = !isfinite((double)acc);
        }
        u[e] = acc;
    }
    if (check) {
        d = wave_max(isnan(d) ? 0.0 : d);
        a = wave_max(isnan(a) ? 0.0 : a);
        bad = wave_or(bad);
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&R.resid[b], (unsigned long long)__double_as_longlong(d));
            atomicMax(&R.maxabs[b], (unsigned long long)__double_as_longlong(a));
            if (bad) atomicOr(&R.bad[b], 1);
        }
    }
}

// ======================================================================
// Fused back-end: one workgroup per solve, both species resident in LDS as
// u[2][N][N+1] (padded rows).  The workgroup runs its solve by itself: at
// every evaluation step (a multiple of check_every, or max_steps) it keeps
// the previous state in HBM, takes the step, computes the FP64 residual
// max |u^s - u^{s-1}| / dt, max |u| and a non-finite flag over both species,
// and retires when the stop rule fires.  No host round trip per step.


template <int N>
__device__ __forceinline__ int lds_addr(int e)
{
    const int c = e / (N * N), rem = e % (N * N);
    return c * (N * (N + 1)) + (rem / N) * (N + 1) + rem % N;
}

// Load the solve, step it with body() (one IMEX step on the LDS state,
// ending with a barrier) until the stop rule fires, store it.
template <typename T, int N, int THREADS, typename Body>
__device__ __forceinline__ void run_solve(T *sm, T *u, int b, double dt, const PersistArgs &pa, Body &&body)
{
    constexpr int WAVES = THREADS / 64;
    __shared__ double red[2 * WAVES];
    __shared__ int s_bad;
    __shared__ int s_stop;
    const int tid = threadIdx.x;
    for (int e = tid; e < 2 * N * N; e += THREADS) sm[lds_addr<N>(e)] = u[e];
    if (tid == 0) s_bad = 0;
    __syncthreads();
    long long step = pa.steps[b];
    while (step < pa.max_steps) {
        const long long next = step + 1;
        const bool eval = (next % pa.check == 0) || (next == pa.max_steps);
        if (eval)
            for (int e = tid; e < 2 * N * N; e += THREADS) u[e] = sm[lds_addr<N>(e)];
        body();
        step = next;
        if (eval) {
            double d = 0.0, a = 0.0;
            int bad = 0;
            for (int e = tid; e < 2 * N * N; e += THREADS) {
                const T nv = sm[lds_addr<N>(e)];
                const double dv = fabs((double)nv - (double)u[e]);
                const double av = fabs((double)nv);
                if (!isfinite((double)nv)) bad = 1;
                d = fmax(d, isnan(dv) ? 0.0 : dv);
                a = fmax(a, isnan(av) ? 0.0 : av);
            }
            d = wave_max(d);
            a = wave_max(a);
            bad = wave_or(bad);
            const int wv = tid / 64;
            if ((tid & 63) == 0) {
                red[wv] = d;
                red[WAVES + wv] = a;
                if (bad) s_bad = 1;
            }
            __syncthreads();
            if (tid == 0) {
                double dm = 0.0, am = 0.0;
                for (int w = 0; w < WAVES; ++w) {
                    dm = fmax(dm, red[w]);
                    am = fmax(am, red[WAVES + w]);
                }
                const double r = dm / dt;
                int st = -1;
                if (s_bad) st = CIL_SOLVE_NONFINITE;
                else if (pa.tol > 0.0 && r < pa.tol) st = CIL_SOLVE_OK;
                else if (pa.tol > 0.0 && pa.floor_coef > 0.0 && r < pa.floor_coef * am) st = CIL_SOLVE_FP32_FLOOR;
                else if (next == pa.max_steps) st = pa.tol > 0.0 ? CIL_SOLVE_MAXSTEPS : CIL_SOLVE_OK;
                pa.resid[b] = s_bad ? (double)NAN : r;
                if (st >= 0) pa.status[b] = st;
                s_stop = st >= 0;
            }
            __syncthreads();
            if (s_stop) break;
        }
    }
    for (int e = tid; e < 2 * N * N; e += THREADS) u[e] = sm[lds_addr<N>(e)];
    if (tid == 0) pa.steps[b] = step;
}

// Line variant: 2N threads, thread t handles species t / N, line t % N,
// whole line in its registers (dct_reg.hpp).
template <typename T, int N>
__global__ __launch_bounds__(2 * N) void k_fused(const DevSolve *S, const int *list, T *state, const T *tables,
                                                 int model, double dt, PersistArgs pa)
{
    using D = DctLine<T, N>;
    constexpr int LD = N + 1, SP = N * LD, THREADS = 2 * N;
    __shared__ T sm[2 * SP];
    const int b = list[blockIdx.x];
    const DevSolve s = S[b];
    T *u = state + s.off;
    const T *tab = tables + (size_t)s.tab * 2 * N * N;
    const int tid = threadIdx.x;
    const int sp = tid / N, ln = tid % N;
    T p[4] = {T(s.p[0]), T(s.p[1]), T(s.p[2]), T(s.p[3])};
    const T tdt = T(dt);
    T *ms = sm + sp * SP;
    run_solve<T, N, THREADS>(sm, u, b, dt, pa, [&]() {
        dispatch_model(model, [&](auto MD) {        // explicit reaction, pointwise
            for (int q = tid; q < N * N; q += THREADS) {
                const int a = (q / N) * LD + q % N;
                const T v = sm[a], w = sm[SP + a];
                T f, g;
                kinetics<MD>(p, v, w, f, g);
                sm[a] = v + tdt * f;
                sm[SP + a] = w + tdt * g;
            }
        });
        __syncthreads();
        {   // forward DCT along rows
            T x[N], X[N];
#pragma unroll
            for (int j = 0; j < N; ++j) x[j] = ms[ln * LD + j];
            D::forward(x, X);
#pragma unroll
            for (int j = 0; j < N; ++j) ms[ln * LD + j] = X[j];
        }
        __syncthreads();
        {   // forward along columns, spectral divide, inverse along columns
            T x[N], X[N];
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = ms[i * LD + ln];
            D::forward(x, X);
            const T *tb = tab + (size_t)sp * N * N + ln;
#pragma unroll
            for (int k = 0; k < N; ++k) X[k] *= tb[k * N];
            D::inverse(X, x);
#pragma unroll
            for (int i = 0; i < N; ++i) ms[i * LD + ln] = x[i];
        }
        __syncthreads();
        {   // inverse along rows
            T x[N], X[N];
#pragma unroll
            for (int j = 0; j < N; ++j) X[j] = ms[ln * LD + j];
            D::inverse(X, x);
#pragma unroll
            for (int j = 0; j < N; ++j) ms[ln * LD + j] = x[j];
        }
        __syncthreads();
    });
}

// Second-order line variant (semi-implicit BDF2): as k_fused, with the
// history u^{s-2}, F(u^{s-2}) resident in LDS beside the state.  The first
// step of the launch is the IMEX-Euler step (tables tabE, built with dt);
// later steps take r = (4 u^{s-1} - u^{s-2}) / 3 + (2 dt / 3)(2 F(u^{s-1}) -
// F(u^{s-2})) and the diffusion solve with 2 dt / 3 (tables tabB).
template <typename T, int N>
__global__ __launch_bounds__(2 * N) void k_fused_sbdf2(const DevSolve *S, const int *list, T *state, const T *tabE,
                                                       const T *tabB, int model, double dt, PersistArgs pa)
{
    using D = DctLine<T, N>;
    constexpr int LD = N + 1, SP = N * LD, THREADS = 2 * N;
    __shared__ T sm[6 * SP];                       // state [2][N][N+1], then u^{s-2}, then F(u^{s-2})
    T *uh = sm + 2 * SP, *fh = sm + 4 * SP;
    const int b = list[blockIdx.x];
    const DevSolve s = S[b];
    T *u = state + s.off;
    const size_t toff = (size_t)s.tab * 2 * N * N;
    const int tid = threadIdx.x;
    const int sp = tid / N, ln = tid % N;
    T p[4] = {T(s.p[0]), T(s.p[1]), T(s.p[2]), T(s.p[3])};
    const T tdt = T(dt), c23 = T(2.0 * dt / 3.0), third = T(1.0 / 3.0);   // a multiply, not a divide
    T *ms = sm + sp * SP;
    bool first = true;
    run_solve<T, N, THREADS>(sm, u, b, dt, pa, [&]() {
        dispatch_model(model, [&](auto MD) {        // reaction stage, pointwise
            for (int q = tid; q < N * N; q += THREADS) {
                const int a = (q / N) * LD + q % N;
                const T v = sm[a], w = sm[SP + a];
                T f, g;
                kinetics<MD>(p, v, w, f, g);
                if (first) {
                    sm[a] = v + tdt * f;
                    sm[SP + a] = w + tdt * g;
                } else {
                    sm[a] = (T(4) * v - uh[a]) * third + c23 * (T(2) * f - fh[a]);
                    sm[SP + a] = (T(4) * w - uh[SP + a]) * third + c23 * (T(2) * g - fh[SP + a]);
                }
                uh[a] = v;
                uh[SP + a] = w;
                fh[a] = f;
                fh[SP + a] = g;
            }
        });
        __syncthreads();
        {   // forward DCT along rows
            T x[N], X[N];
#pragma unroll
            for (int j = 0; j < N; ++j) x[j] = ms[ln * LD + j];
            D::forward(x, X);
#pragma unroll
            for (int j = 0; j < N; ++j) ms[ln * LD + j] = X[j];
        }
        __syncthreads();
        {   // forward along columns, spectral divide, inverse along columns
            T x[N], X[N];
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = ms[i * LD + ln];
            D::forward(x, X);
            const T *tb = (first ? tabE : tabB) + toff + (size_t)sp * N * N + ln;
#pragma unroll
            for (int k = 0; k < N; ++k) X[k] *= tb[k * N];
            D::inverse(X, x);
#pragma unroll
            for (int i = 0; i < N; ++i) ms[i * LD + ln] = x[i];
        }
        __syncthreads();
        {   // inverse along rows
            T x[N], X[N];
#pragma unroll
            for (int j = 0; j < N; ++j) X[j] = ms[ln * LD + j];
            D::inverse(X, x);
#pragma unroll
            for (int j = 0; j < N; ++j) ms[ln * LD + j] = x[j];
        }
        __syncthreads();
        first = false;
    });
}

// Spectral tables for the fused back-end:
// tab[s][k][l] = 1 / (4 N^2 (1 + dt nu_s (lam_k + lam_l) / h^2)), in FP64 then T.
template <typename T>
__global__ void k_make_tables(const TabSpec *specs, int ntab, int n, double dt, T *out)
{
    const int t = blockIdx.y;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntab || e >= 2 * n * n) return;
    const int sp = e / (n * n), k = (e / n) % n, l = e % n;
    const TabSpec ts = specs[t];
    const double sk = sinpi((double)k / (2.0 * n)), sl = sinpi((double)l / (2.0 * n));
    const double lam = 4.0 * (sk * sk + sl * sl) * ts.inv_h2;
    const double nu = sp ? ts.nu1 : ts.nu0;
    out[(size_t)t * 2 * n * n + e] = T(1.0 / (4.0 * n * (double)n * (1.0 + dt * nu * lam)));
}

// Quad-variant table: the column pass applies the divisor in the split
// step's V form.  With Y = X_k - i X_{N-k} = ph V (ph = exp(-i pi k / 2N)),
// dividing X_k by D_k and X_{N-k} by D_{N-k} is Y' = S Y + Delta conj(Y),
// S = (D_k + D_{N-k}) / 2, Delta = (D_k - D_{N-k}) / 2, so
// V' = S V + Delta exp(i pi k / N) conj(V):
//   Re V' = A Re V + Ci Im V,  Im V' = B Im V + Ci Re V,
//   A = S + Delta cos(pi k/N), B = S - Delta cos(pi k/N), Ci = Delta sin(pi k/N).
// k = 0 keeps only Re V (X_N does not exist): A = D_0, B = Ci = 0.  Row k = M
// of plane A holds D_M (X_M is carried as a real value).
// Layout: vt[t][s][plane A|B|Ci][k = 0..M][l], M = n/2 (D indexed as tab above).
template <typename T>
__global__ void k_make_vtables(const TabSpec *specs, int ntab, int n, double dt, T *out)
{
    const int t = blockIdx.y;
    const int M = n / 2, rows = M + 1;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntab || e >= 2 * rows * n) return;
    const int sp = e / (rows * n), k = (e / n) % rows, l = e % n;
    const TabSpec ts = specs[t];
    const double nu = sp ? ts.nu1 : ts.nu0;
    auto D = [&](int kk) {
        const double sk = sinpi((double)kk / (2.0 * n)), sl = sinpi((double)l / (2.0 * n));
        const double lam = 4.0 * (sk * sk + sl * sl) * ts.inv_h2;
        return 1.0 / (4.0 * n * (double)n * (1.0 + dt * nu * lam));
    };
    double A, B = 0.0, C = 0.0;
    if (k == 0 || k == M) {
        A = D(k);
    } else {
        const double dk = D(k), dn = D(n - k);
        const double S = 0.5 * (dk + dn), Dl = 0.5 * (dk - dn);
        double sn, cs;
        sincospi((double)k / n, &sn, &cs);
        A = S + Dl * cs;
        B = S - Dl * cs;
        C = Dl * sn;
    }
    T *o = out + (size_t)t * 2 * 3 * rows * n + (size_t)sp * 3 * rows * n + (size_t)k * n + l;
    o[0] = T(A);
    o[(size_t)rows * n] = T(B);
    o[(size_t)2 * rows * n] = T(C);
}

template <typename S, typename D>
__global__ void k_convert_solves(const DevSolve *Ssrc, const DevSolve *Sdst, const int *list,
                                 const S *src, D *dst)
{
    const int b = list[blockIdx.y];
    const DevSolve a = Ssrc[b], c = Sdst[b];
    const int sz = 2 * a.n * a.n;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < sz; e += gridDim.x * blockDim.x)
        dst[c.off + e] = D(src[a.off + e]);
}

// ======================================================================
// Host side.

namespace {

struct PlainTables {
    void *C = nullptr, *Ct = nullptr, *Cw = nullptr;   // T[n*n]
    double *lam = nullptr;                              // double[n]
};
std::map<std::tuple<int, int, int>, PlainTables> g_plain_tables;   // (device, n, is_f32)

template <typename T>
int plain_tables(int n, PlainTables *out)
{
    int dev;
    CIL_TRY(current_device(&dev));
    auto key = std::make_tuple(dev, n, (int)std::is_same<T, float>::value);
    auto it = g_plain_tables.find(key);
    if (it != g_plain_tables.end()) {
        *out = it->second;
        return CIL_OK;
    }
    std::vector<T> C(n * n), Ct(n * n), Cw(n * n);
    std::vector<double> lam(n);
    for (int k = 0; k < n; ++k) {
        const double wk = (k == 0 ? 1.0 : 2.0) / n;
        for (int j = 0; j < n; ++j) {
            const double c = std::cos(M_PI * k * (2.0 * j + 1.0) / (2.0 * n));
            C[k * n + j] = T(c);
            Ct[j * n + k] = T(c);
            Cw[k * n + j] = T(wk * c);
        }
        const double sk = std::sin(M_PI * k / (2.0 * n));
        lam[k] = 4.0 * sk * sk;
    }
    PlainTables t;
    size_t bytes = sizeof(T) * n * n;
    if (hipMalloc(&t.C, bytes) != hipSuccess || hipMalloc(&t.Ct, bytes) != hipSuccess ||
        hipMalloc(&t.Cw, bytes) != hipSuccess || hipMalloc(&t.lam, sizeof(double) * n) != hipSuccess)
        return set_error(CIL_ENOMEM, "table allocation failed");
    CIL_HIP(hipMemcpy(t.C, C.data(), bytes, hipMemcpyHostToDevice));
    CIL_HIP(hipMemcpy(t.Ct, Ct.data(), bytes, hipMemcpyHostToDevice));
    CIL_HIP(hipMemcpy(t.Cw, Cw.data(), bytes, hipMemcpyHostToDevice));
    CIL_HIP(hipMemcpy(t.lam, lam.data(), sizeof(double) * n, hipMemcpyHostToDevice));
    g_plain_tables[key] = t;
    *out = t;
    return CIL_OK;
}

// Auxiliary streams (default priority) for running the persistent kernels of
// different grid sides side by side, and fork/join events.  A call leases a set
// for as long as it runs (calls of several threads at once have one each: a shared
// fork event would be recorded anew between another call's record and its waits)
// and gives it back; up to kKept sets stay per device.
constexpr size_t kKept = 8;
std::mutex g_lease_mu;
struct AuxStreams {
    std::vector<hipStream_t> st;
    std::vector<hipEvent_t> ev;     // ev[0] fork, ev[1 + g] join of stream g
    ~AuxStreams()
    {
        for (hipStream_t s : st) (void)hipStreamDestroy(s);
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    }
};
// device -> sets not in use (never destroyed: the runtime may be gone by then)
auto &g_aux = *new std::map<int, std::vector<std::unique_ptr<AuxStreams>>>;

struct AuxLease {
    std::unique_ptr<AuxStreams> set;
    int dev = 0;
    ~AuxLease()
    {
        if (!set) return;
        std::lock_guard<std::mutex> lk(g_lease_mu);
        if (g_aux[dev].size() < kKept) g_aux[dev].push_back(std::move(set));
    }
    int take(int streams, int joins)
    {
        CIL_TRY(current_device(&dev));
        {
            std::lock_guard<std::mutex> lk(g_lease_mu);
            auto &free_sets = g_aux[dev];
            if (!free_sets.empty()) {
                set = std::move(free_sets.back());
                free_sets.pop_back();
            }
        }
        if (!set) set.reset(new AuxStreams);
        while ((int)set->st.size() < streams) {
            hipStream_t s;
            CIL_HIP(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
            set->st.push_back(s);
        }
        while ((int)set->ev.size() < joins + 1) {
            hipEvent_t e;
            CIL_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
            set->ev.push_back(e);
        }
        return CIL_OK;
    }
};

// Pinned blocks that results come back through, leased likewise: one that a call
// has not read yet is no other call's.
std::map<int, std::multimap<size_t, void *>> g_stage;              // device -> (capacity, block) not in use
struct StageLease {
    void *p = nullptr;
    size_t cap = 0;
    int dev = 0;
    ~StageLease()
    {
        if (!p) return;
        void *drop = nullptr;
        {
            std::lock_guard<std::mutex> lk(g_lease_mu);
            auto &m = g_stage[dev];
            m.emplace(cap, p);
            if (m.size() > kKept) {                      // the smallest goes
                drop = m.begin()->second;
                m.erase(m.begin());
            }
        }
        if (drop) (void)hipHostFree(drop);
    }
    int take(size_t bytes)
    {
        CIL_TRY(current_device(&dev));
        {
            std::lock_guard<std::mutex> lk(g_lease_mu);
            auto &m = g_stage[dev];
            auto it = m.lower_bound(bytes);
            if (it != m.end()) {
                cap = it->first;
                p = it->second;
                m.erase(it);
                return CIL_OK;
            }
        }
        cap = std::max<size_t>(64 * 1024, bytes + bytes / 4);
        if (hipHostMalloc(&p, cap, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            p = nullptr;
            return set_error(CIL_ENOMEM, "pinned host buffer of %zu bytes failed", cap);
        }
        return CIL_OK;
    }
};

// How a persistent group runs: one lane or a quad of lanes per grid line, or
// the matrix cores.
enum FusedKind { KIND_LINE = 0, KIND_QUAD, KIND_MM };

int fused_supported(int n, bool f32)
{
    return f32 ? (n == 32 || n == 64 || n == 128) : (n == 32 || n == 64);
}

int g_quad_shape_option = -1;
int g_polish_separate = 0;         // 1: the polish always in a launch of its own
// 0: off, else the base of the priority levels.  Measured on the 500-solve GM
// batch (FP64, residual 1e-8): off 30.5 ms; base 3: 30.2; 10: 29.9; 100: 29.5;
// 1000: 29.4.
double g_wave_priority = 100.0;

// The kernel a path selects.  AUTO and FUSED run on the matrix cores, which
// measured faster than the quad-lane kernels at every side and batch size (us
// per step, matrix cores / quad: 128 FHN 32^2 solves FP32 1.03 / 2.12, FP64
// 1.63 / 2.95; one 64^2 solve FP32 3.4 / 6.3, FP64 5.7 / 11.4, 512 of them 7.2 /
// 9.7 and 12.4 / 17.7; 256 128^2 solves FP32 14.1 / 21.2); a quad-lane code
// shape chosen by option keeps the quad kernel.
FusedKind fused_kind(int path)
{
    if (path == CIL_PATH_FUSED_LINE) return KIND_LINE;
    if (path == CIL_PATH_FUSED_QUAD || g_quad_shape_option >= 0) return KIND_QUAD;
    return KIND_MM;
}

// Whether side n has a persistent kernel on this path.  AUTO takes the matrix
// cores for any side whose field fits the LDS (192 FP64 solves of sides 20 to
// 96: 34 us a step against 378 for the plain path); an explicit path, and a
// quad-lane code shape chosen by option, have the sides they name.
bool persistent_supported(int n, bool f32, int path)
{
    if (path == CIL_PATH_PLAIN) return false;
    if (fused_supported(n, f32)) return true;
    return path == CIL_PATH_AUTO && g_quad_shape_option < 0 && n >= 2 && n <= mm_max_side(f32);
}

// Whether a side that has both a persistent and a tile-by-tile kernel takes the
// latter: while all solves of the call together are few wavefronts for the
// chip's 1024 SIMDs, and the evaluation steps, at which the host looks, are
// some steps apart.  us per step, tile by tile / persistent (FHN):
//   FP64 96^2        1 solve 16.0 / 28.9, 32 20.9 / 31.2, 64 24.0 / 31.6, 128 37.9 /
//                    32.8; 16 solves evaluated every step 42.6 / 44.4, every
//                    second 30.3 / 37.0, 64 every second 38.9 / 37.2, every third
//                    32.8 / 34.7; 128 of sides 64, 51, 70 25.5 / 31.8, 256 37.7 / 33.0
//   FP32 112^2       1 solve 16.4 / 38.0, 64 25.5 / 40.9, 128 40.0 / 41.0, 192 52 / 42
//   FP32 96^2        1 solve 12.0 / 15.8, 32 16.7 / 18.2, 48 17.2 / 18.1, 64 18.7 / 18.1
//   FP32 128^2       1 solve 10.5 / 14.4, 32 15.4 / 16.5, 48 17.4 / 16.4
bool tile_by_tile(int n, bool f32, int64_t waves, int check)
{
    if (!split_supported(n)) return false;
    if (f32 && (n <= 96 || n == 128)) return waves <= 512 && check >= 8;
    return waves <= (f32 ? 1900 : 1200) && check >= 3;
}

int quad_shape(bool f32, int n)
{
    if (g_quad_shape_option >= 0) return g_quad_shape_option;
    // Measured on MI355X with the plans' autotuner (completion time of whole
    // batches): 32^2 runs fastest with one species per lane (128 FHN solves:
    // FP32 12.2 ms against 18.3 for both species per lane, FP64 16.2 against
    // 24.6); 64^2 and 128^2 with both species per lane, where the V-form
    // divisor pays in FP32 but not in FP64 (500 GM 64^2 solves in FP64: 30.4
    // ms X-form, 33.6 V-form; its third table plane costs more load latency
    // than it saves operations).
    if (n == 32) return 1;
    return f32 ? 2 : 0;
}

}  // namespace

// Device blocks reused across simulate calls, per device: a call's buffers go
// back to this pool instead of hipFree, so repeated calls of similar size
// allocate nothing.  Freed by cil_shutdown.
std::mutex g_pool_mu;
std::map<int, std::multimap<size_t, void *>> g_pool;     // device -> (capacity, block)

size_t pool_capacity(size_t bytes)
{
    if (bytes <= ((size_t)1 << 20)) {
        size_t c = 256;
        while (c < bytes) c <<= 1;
        return c;
    }
    return (bytes + ((size_t)1 << 20) - 1) & ~(((size_t)1 << 20) - 1);
}

// Library-owned stepper resources (cached DCT matrices of the plain path,
// auxiliary streams and events, the pool of call buffers), freed by
// cil_shutdown.
int stepper_release()
{
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (auto &kv : g_plain_tables) {
        (void)hipSetDevice(std::get<0>(kv.first));
        (void)hipFree(kv.second.C);
        (void)hipFree(kv.second.Ct);
        (void)hipFree(kv.second.Cw);
        (void)hipFree(kv.second.lam);
    }
    g_plain_tables.clear();
    {
        std::lock_guard<std::mutex> lk(g_lease_mu);
        for (auto &kv : g_aux) {
            (void)hipSetDevice(kv.first);
            kv.second.clear();
        }
        for (auto &kv : g_stage) {
            for (auto &b : kv.second) (void)hipHostFree(b.second);
            kv.second.clear();
        }
    }
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        for (auto &kv : g_pool) {
            (void)hipSetDevice(kv.first);
            for (auto &b : kv.second) (void)hipFree(b.second);
        }
        g_pool.clear();
    }
    (void)hipSetDevice(cur);
    return CIL_OK;
}

int set_polish_separate(int64_t v)
{
    if (v != 0 && v != 1) return set_error(CIL_EINVAL, "polish option must be 0 or 1");
    g_polish_separate = (int)v;
    return CIL_OK;
}

int set_wave_priority(int64_t v)
{
    if (v < 0 || v == 1 || v > 1000000) return set_error(CIL_EINVAL, "wave priority option must be 0 or in [2, 1e6]");
    g_wave_priority = (double)v;
    return CIL_OK;
}

int set_quad_shape(int64_t v)
{
    if (v < -1 || v >= kQuadShapes) return set_error(CIL_EINVAL, "quad shape %lld out of range", (long long)v);
    g_quad_shape_option = (int)v;
    return CIL_OK;
}

namespace {

// Matrix-core launch; the kernel's name in the profiler goes by side where the
// side has a kernel of its own.
template <typename T>
int launch_mm_named(int n, int scheme, int nl, const DevSolve *S, const int *list, T *state, const T *tab,
                    const T *tab2, const T *cst, int model, double dt, const PersistArgs &pa, hipStream_t st)
{
    static const char *names[2][2][4] = {
        {{"k_mm_f64", "k_mm_f64_n32", "k_mm_f64_n64", "k_mm_f64_n128"},
         {"k_mm_f32", "k_mm_f32_n32", "k_mm_f32_n64", "k_mm_f32_n128"}},
        {{"k_mm_sbdf2_f64", "k_mm_sbdf2_f64_n32", "k_mm_sbdf2_f64_n64", "k_mm_sbdf2_f64_n128"},
         {"k_mm_sbdf2_f32", "k_mm_sbdf2_f32_n32", "k_mm_sbdf2_f32_n64", "k_mm_sbdf2_f32_n128"}}};
    const char *name = names[scheme][sizeof(T) == 4][n == 32 ? 1 : n == 64 ? 2 : n == 128 ? 3 : 0];
    const ProfMark pm = prof_begin(name, st);
    const int rc = launch_mm<T>(n, scheme, nl, S, list, state, tab, tab2, cst, model, dt, pa, st);
    prof_end(pm, st);
    if (rc) return set_error(rc, "no matrix-core kernel for n = %d", n);
    return check_launch(name);
}

template <typename T>
int launch_persistent(int n, bool quad, int shape, int nl, const DevSolve *S, const int *list, T *state, const T *tables,
                      int model, double dt, const PersistArgs &pa, hipStream_t st)
{
    const bool f32 = std::is_same<T, float>::value;
    const int ni = n == 32 ? 0 : (n == 64 ? 1 : 2);
    static const char *nq32[3] = {"k_fused_q_f32_n32", "k_fused_q_f32_n64", "k_fused_q_f32_n128"};
    static const char *nq64[3] = {"k_fused_q_f64_n32", "k_fused_q_f64_n64", "k_fused_q_f64_n128"};
    static const char *nl32[3] = {"k_fused_f32_n32", "k_fused_f32_n64", "k_fused_f32_n128"};
    static const char *nl64[3] = {"k_fused_f64_n32", "k_fused_f64_n64", "k_fused_f64_n128"};
    const char *name = quad ? (f32 ? nq32[ni] : nq64[ni]) : (f32 ? nl32[ni] : nl64[ni]);
    if (!f32 && n == 128) return set_error(CIL_EUNSUPPORTED, "fused FP64 stepper supports n = 32, 64");
    const ProfMark pm = prof_begin(name, st);
    if (quad) {
        const int rc = f32 ? launch_quad_f32(n, shape, nl, S, list, (float *)state, (const float *)tables, model, dt, pa, st)
                           : launch_quad_f64(n, shape, nl, S, list, (double *)state, (const double *)tables, model, dt,
                                             pa, st);
        if (rc) return set_error(rc, "no fused quad kernel for n = %d", n);
    } else {
        if (n == 32)
            hipLaunchKernelGGL((k_fused<T, 32>), dim3(nl), dim3(64), 0, st, S, list, state, tables, model, dt, pa);
        else if (n == 64)
            hipLaunchKernelGGL((k_fused<T, 64>), dim3(nl), dim3(128), 0, st, S, list, state, tables, model, dt, pa);
        else if constexpr (std::is_same<T, float>::value)
            hipLaunchKernelGGL((k_fused<T, 128>), dim3(nl), dim3(256), 0, st, S, list, state, tables, model, dt, pa);
    }
    prof_end(pm, st);
    return check_launch(name);
}

// One plain group: solves with one grid side n, advanced in lockstep; or the
// solves of any sides that step tile by tile on the matrix cores (split).
template <typename T>
struct PlainGroup {
    int n = 0;
    std::vector<int> active;
    int *dlist = nullptr;
    void *work = nullptr;         // 2 buffers [cap][2][n][n]
    size_t work_cap = 0;
    bool split = false;
    std::vector<std::vector<SplitItem<T>>> tiles;    // per active solve
    std::vector<SplitItem<T>> items;              // in launch order
    SplitItem<T> *ditems = nullptr;
    T *c0 = nullptr, *ct = nullptr;
};

// History of the second-order stepper for one plain launch: u^{s-2} and
// F(u^{s-2}) in the state's layout, and the step index the launch starts at.
template <typename T>
struct Sbdf2Args {
    T *uh, *fh;
    int64_t step0;
};

template <typename T>
int launch_plain(PlainGroup<T> &g, const DevSolve *S, T *u, int nl, int model, double dt, int K, StepResults R,
                 hipStream_t st, const Sbdf2Args<T> *bdf = nullptr)
{
    PlainTables tb;
    CIL_TRY(plain_tables<T>(g.n, &tb));
    const int n = g.n, N2 = n * n;
    T *A = (T *)g.work;
    T *Bw = A + g.work_cap * 2 * N2;
    const dim3 blk(256);
    const dim3 grid1((N2 + 255) / 256, nl), grid2((2 * N2 + 255) / 256, nl);
    const bool f32 = std::is_same<T, float>::value;
    const ProfMark pm = prof_begin(bdf ? (f32 ? "plain_step_sbdf2_f32" : "plain_step_sbdf2_f64")
                                       : (f32 ? "plain_step_f32" : "plain_step_f64"), st);
    for (int k = 0; k < K; ++k) {
        const int check = (k == K - 1);
        double dts = dt;                   // the diffusion solve's step
        if (bdf) {
            const int first = (bdf->step0 + k == 0);
            if (!first) dts = 2.0 * dt / 3.0;
            hipLaunchKernelGGL(k_plain_reaction_sbdf2<T>, grid1, blk, 0, st, S, g.dlist, u, A, bdf->uh, bdf->fh, n,
                               model, dt, first);
        } else {
            hipLaunchKernelGGL(k_plain_reaction<T>, grid1, blk, 0, st, S, g.dlist, u, A, n, model, dt);
        }
        hipLaunchKernelGGL(k_plain_rows_fwd<T>, grid2, blk, 0, st, g.dlist, A, Bw, (const T *)tb.Ct, n);
        hipLaunchKernelGGL(k_plain_cols_fwd_div<T>, grid2, blk, 0, st, S, g.dlist, Bw, A, (const T *)tb.C, tb.lam, n,
                           dts);
        hipLaunchKernelGGL(k_plain_cols_inv<T>, grid2, blk, 0, st, g.dlist, A, Bw, (const T *)tb.Cw, n);
        hipLaunchKernelGGL(k_plain_rows_inv<T>, grid2, blk, 0, st, S, g.dlist, Bw, u, (const T *)tb.Cw, n, check, R);
    }
    prof_end(pm, st);
    return check_launch("plain stepper");
}

}  // namespace

// Device buffers owned by one simulate call (returned to the pool at its end;
// a call that did not reach its final synchronisation first waits for the
// device, so no block goes back while queued work may still use it).
struct CallBuffers {
    struct Block {
        void *p;
        size_t cap;
        int dev;
    };
    std::vector<Block> blocks;
    bool done = false;
    ~CallBuffers()
    {
        if (blocks.empty()) return;
        if (!done) (void)hipDeviceSynchronize();
        std::lock_guard<std::mutex> lk(g_pool_mu);
        for (const Block &b : blocks) g_pool[b.dev].emplace(b.cap, b.p);
    }
    int alloc(void **p, size_t bytes)
    {
        int dev;
        CIL_TRY(current_device(&dev));
        const size_t cap = pool_capacity(bytes == 0 ? 16 : bytes);
        {
            std::lock_guard<std::mutex> lk(g_pool_mu);
            auto &m = g_pool[dev];
            auto it = m.lower_bound(cap);
            if (it != m.end() && it->first <= 2 * cap) {
                *p = it->second;
                blocks.push_back(Block{it->second, it->first, dev});
                m.erase(it);
                return CIL_OK;
            }
        }
        if (hipMalloc(p, cap) != hipSuccess) {
            (void)hipGetLastError();
            return set_error(CIL_ENOMEM, "device allocation of %zu bytes failed", cap);
        }
        blocks.push_back(Block{*p, cap, dev});
        return CIL_OK;
    }
};

namespace {

struct SimCtx {
    int model;
    double dt, tol;
    int64_t max_steps;
    int check;
    double floor_coef32;          // FP32 floor per unit max|u| (0 if no floor test)
    hipStream_t st;
    CallBuffers *cb;
    std::vector<int64_t> steps;   // per solve (host)
    std::vector<double> fres;
    std::vector<int> status;
    std::vector<int64_t> sw;      // mixed launches: step of the FP32 -> FP64 switch (-1: not a mixed solve)
    int polish = 0;               // 0 none, 1 FP64 steps, 2 refinement form (FP32 calls)
    int scheme = 0;               // 0 IMEX Euler, 1 second-order IMEX (plain back-end)
    void *uh = nullptr, *fh = nullptr;   // second-order history, state layout
};

// FP32 -> FP64 within one launch (k_fused_q_mixed) for these grid sides.
struct MixedArgs {
    double *state64;              // FP64 snapshots or FP64 state, same element layout as the FP32 state
    long long *sw;                // per solve: switch step
    int refine;                   // 1: the continuation is the refinement form, else FP64 steps
};

bool mixed_supported(int n, FusedKind kind)
{
    return kind != KIND_LINE && g_quad_shape_option < 0 && (n == 32 || n == 64);
}

// Spectral tables for the solves in `ids` (side n): one per distinct (h, nu);
// sets hs[b].tab.  make_specs uploads the distinct ones, make_tables and
// make_mm_tables build from them.
int make_specs(SimCtx &c, const std::vector<int> &ids, std::vector<DevSolve> &hs, void **dspecs, int *count)
{
    std::map<std::tuple<double, double, double>, int> uniq;
    std::vector<TabSpec> specs;
    for (int b : ids) {
        auto key = std::make_tuple(hs[b].inv_h2, hs[b].nu[0], hs[b].nu[1]);
        auto it = uniq.find(key);
        if (it == uniq.end()) {
            it = uniq.emplace(key, (int)specs.size()).first;
            specs.push_back(TabSpec{hs[b].inv_h2, hs[b].nu[0], hs[b].nu[1]});
        }
        hs[b].tab = it->second;
    }
    *count = (int)specs.size();
    CIL_TRY(c.cb->alloc(dspecs, sizeof(TabSpec) * specs.size()));
    CIL_HIP(hipMemcpyAsync(*dspecs, specs.data(), sizeof(TabSpec) * specs.size(), hipMemcpyHostToDevice, c.st));
    return CIL_OK;
}

template <typename T>
int make_tables(SimCtx &c, int n, const std::vector<int> &ids, std::vector<DevSolve> &hs, void **tables, bool vform,
                double dt_tab = 0.0)
{
    const double dtt = dt_tab > 0.0 ? dt_tab : c.dt;
    void *dspecs;
    int count;
    CIL_TRY(make_specs(c, ids, hs, &dspecs, &count));
    if (vform) {
        const size_t per = (size_t)2 * 3 * (n / 2 + 1) * n;
        CIL_TRY(c.cb->alloc(tables, sizeof(T) * per * count));
        dim3 grid((unsigned)((2 * (n / 2 + 1) * n + 255) / 256), (unsigned)count);
        hipLaunchKernelGGL(k_make_vtables<T>, grid, dim3(256), 0, c.st, (const TabSpec *)dspecs, count, n, dtt,
                           (T *)*tables);
        return check_launch("k_make_vtables");
    }
    CIL_TRY(c.cb->alloc(tables, sizeof(T) * (size_t)2 * n * n * count));
    dim3 grid((2 * n * n + 255) / 256, (unsigned)count);
    hipLaunchKernelGGL(k_make_tables<T>, grid, dim3(256), 0, c.st, (const TabSpec *)dspecs, count, n, dtt,
                       (T *)*tables);
    return check_launch("k_make_tables");
}

// The matrix-core stepper's divisors (second != nullptr: a second set for the
// second-order scheme's later steps, dt2) and, for sides without a folding of
// their own, its constant blocks.
struct MmTables {
    void *tab = nullptr, *tab2 = nullptr, *cst = nullptr;
};
template <typename T>
int make_mm_tables(SimCtx &c, int n, const std::vector<int> &ids, std::vector<DevSolve> &hs, MmTables *out,
                   double dt2 = 0.0)
{
    void *dspecs;
    int count;
    CIL_TRY(make_specs(c, ids, hs, &dspecs, &count));
    const size_t bytes = sizeof(T) * mm_table_elems(n) * count;
    CIL_TRY(c.cb->alloc(&out->tab, bytes));
    CIL_TRY(mm_make_tables<T>(n, (const TabSpec *)dspecs, count, c.dt, (T *)out->tab, c.st));
    if (dt2 > 0.0) {
        CIL_TRY(c.cb->alloc(&out->tab2, bytes));
        CIL_TRY(mm_make_tables<T>(n, (const TabSpec *)dspecs, count, dt2, (T *)out->tab2, c.st));
    }
    if (mm_const_elems(n)) {
        CIL_TRY(c.cb->alloc(&out->cst, sizeof(T) * mm_const_elems(n)));
        CIL_TRY(mm_make_consts<T>(n, (T *)out->cst, c.st));
    }
    return CIL_OK;
}

// Per-solve results of fused launches (steps, last residual, status and, for
// mixed launches, the switch step) back to the host: pinned staging, so the
// copies are queued without blocking, and one wait.
struct HostResults {
    StageLease block;                     // (what the pointers point into)
    const long long *steps;
    const double *res;
    const int *stat;
    const long long *sw;
};
int fetch_results(SimCtx &c, int B, const long long *dsteps, const double *dres, const int *dstat,
                  const long long *dsw, HostResults *out)
{
    const size_t b8 = sizeof(long long) * (size_t)B;
    CIL_TRY(out->block.take(3 * b8 + sizeof(int) * (size_t)B));
    char *const hb = (char *)out->block.p;
    out->steps = (const long long *)hb;
    out->res = (const double *)(hb + b8);
    out->sw = dsw ? (const long long *)(hb + 2 * b8) : nullptr;
    out->stat = (const int *)(hb + 3 * b8);
    CIL_HIP(hipMemcpyAsync(hb, dsteps, b8, hipMemcpyDeviceToHost, c.st));
    CIL_HIP(hipMemcpyAsync(hb + b8, dres, b8, hipMemcpyDeviceToHost, c.st));
    CIL_HIP(hipMemcpyAsync(hb + 3 * b8, dstat, sizeof(int) * (size_t)B, hipMemcpyDeviceToHost, c.st));
    if (dsw) CIL_HIP(hipMemcpyAsync(hb + 2 * b8, dsw, b8, hipMemcpyDeviceToHost, c.st));
    return stream_wait(c.st);
}

// FP64 tables of the FP64-step polish, and the mixed launch, for either kind of
// kernel.  mode as launch_quad_mixed's.
int polish_tables(SimCtx &c, int n, const std::vector<int> &ids, std::vector<DevSolve> &hs, FusedKind kind, void **tab)
{
    if (kind != KIND_MM) return make_tables<double>(c, n, ids, hs, tab, kQuadShape[quad_shape(false, n)].vform);
    MmTables mt;
    CIL_TRY(make_mm_tables<double>(c, n, ids, hs, &mt));
    *tab = mt.tab;
    return CIL_OK;
}

int launch_mixed_named(FusedKind kind, int n, int nl, const DevSolve *S, const int *list, float *state,
                       double *state64, const float *tab32, const double *tab64, int model, double dt,
                       const PersistArgs &pa32, const PersistArgs &pa64, long long *sw, int refine, int mode,
                       hipStream_t st)
{
    static const char *names[2][2][3] = {
        {{"k_fused_q_mixed_n32", "k_fused_q_mixed_n32_phase1", "k_fused_q_mixed_n32_phase2"},
         {"k_fused_q_mixed_n64", "k_fused_q_mixed_n64_phase1", "k_fused_q_mixed_n64_phase2"}},
        {{"k_mm_mixed_n32", "k_mm_mixed_n32_phase1", "k_mm_mixed_n32_phase2"},
         {"k_mm_mixed_n64", "k_mm_mixed_n64_phase1", "k_mm_mixed_n64_phase2"}}};
    const char *name = names[kind == KIND_MM][n == 64][mode];
    const ProfMark pm = prof_begin(name, st);
    const int rc = kind == KIND_MM ? launch_mm_mixed(n, nl, S, list, state, state64, tab32, tab64, model, dt, pa32,
                                                     pa64, sw, refine, mode, st)
                                   : launch_quad_mixed(n, nl, S, list, state, state64, tab32, tab64, model, dt, pa32,
                                                       pa64, sw, refine, mode, st);
    prof_end(pm, st);
    if (rc) return set_error(rc, "no mixed-precision kernel for n = %d", n);
    return check_launch(name);
}

// Fused solves, all sides in one go: every workgroup runs its solve from
// steps[b] until its stop rule fires.  `dsteps/dres/dstat` are per-solve
// device arrays; the host copies are refreshed after the launches.  `aside`, if
// given, is called once the kernels run, all on streams of their own, to run
// other solves on the caller's stream beside them.
template <typename T>
int run_fused(SimCtx &c, const std::map<int, std::vector<int>> &byn, std::vector<DevSolve> &hs, DevSolve *dS, T *state,
              FusedKind kind, double floor_coef, long long *dsteps, double *dres, int *dstat,
              const MixedArgs *mx = nullptr, const std::function<int()> *aside = nullptr)
{
    if (byn.empty()) return CIL_OK;
    const bool quad = kind != KIND_LINE;
    std::vector<void *> tabs, tabs64;
    std::vector<MmTables> mms;
    std::vector<char> mixed;
    for (auto &kv : byn) {
        void *t = nullptr, *t64 = nullptr;
        MmTables mt;
        const bool mix = mx && mixed_supported(kv.first, kind);
        if (kind == KIND_MM)
            CIL_TRY(make_mm_tables<T>(c, kv.first, kv.second, hs, &mt, c.scheme ? 2.0 * c.dt / 3.0 : 0.0));
        else
            CIL_TRY(make_tables<T>(c, kv.first, kv.second, hs, &t,
                                   quad && kQuadShape[quad_shape(std::is_same<T, float>::value, kv.first)].vform));
        mms.push_back(mt);
        if (mix && !mx->refine && !g_polish_separate) CIL_TRY(polish_tables(c, kv.first, kv.second, hs, kind, &t64));
        tabs.push_back(t);
        tabs64.push_back(t64);
        mixed.push_back(mix);
    }
    const int B = (int)hs.size();
    CIL_HIP(hipMemcpyAsync(dS, hs.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, c.st));
    std::vector<long long> hsteps(c.steps.begin(), c.steps.end());
    CIL_HIP(hipMemcpyAsync(dsteps, hsteps.data(), sizeof(long long) * B, hipMemcpyHostToDevice, c.st));
    PersistArgs pa{(long long)c.max_steps, c.tol, c.check, floor_coef, dsteps, dres, dstat, g_wave_priority};
    // Several grid sides: each side's persistent kernel on its own stream, the
    // most expensive (n^2 log n x solves) launched first, joined back into the
    // caller's stream, so the call stays ordered on it.
    std::vector<std::pair<double, int>> order;
    {
        int gi = 0;
        for (auto &kv : byn) {
            const double n = kv.first;
            order.push_back({-n * n * std::log2(n) * (double)kv.second.size(), gi++});
        }
        std::sort(order.begin(), order.end());
    }
    std::vector<int *> dls;
    for (auto &kv : byn) {
        int *dl;
        CIL_TRY(c.cb->alloc((void **)&dl, sizeof(int) * kv.second.size()));
        CIL_HIP(hipMemcpyAsync(dl, kv.second.data(), sizeof(int) * kv.second.size(), hipMemcpyHostToDevice, c.st));
        dls.push_back(dl);
    }
    AuxLease lease;
    AuxStreams *aux = nullptr;
    const int ng = (int)byn.size();
    // a side per stream, at most eight streams (a batch may hold a hundred sides; four hardware queues serve them)
    const int nst = std::min(ng, 8);
    if (ng > 1 || aside) {
        CIL_TRY(lease.take(nst, ng));
        aux = lease.set.get();
        CIL_HIP(hipEventRecord(aux->ev[0], c.st));
    }
    std::vector<const std::pair<const int, std::vector<int>> *> groups;
    for (auto &kv : byn) groups.push_back(&kv);
    for (auto &o : order) {
        const int gi = o.second;
        const auto &kv = *groups[gi];
        hipStream_t gst = c.st;
        if (aux) {
            gst = aux->st[gi % nst];
            CIL_HIP(hipStreamWaitEvent(gst, aux->ev[0], 0));
        }
        const int shape = quad_shape(std::is_same<T, float>::value, kv.first);
        if constexpr (std::is_same<T, float>::value) {
            if (mixed[gi]) {
                PersistArgs pa64 = pa;
                pa64.floor_coef = 0.0;
                // separate polish: the FP32 phase here, the continuation in a
                // launch of its own over the solves at their floor (run_phase2)
                const int mode = g_polish_separate ? 1 : 0;
                CIL_TRY(launch_mixed_named(kind, kv.first, (int)kv.second.size(), dS, dls[gi], state, mx->state64,
                                           (const float *)(kind == KIND_MM ? mms[gi].tab : tabs[gi]),
                                           (const double *)tabs64[gi], c.model, c.dt, pa, pa64, mx->sw, mx->refine,
                                           mode, gst));
                if (aux) CIL_HIP(hipEventRecord(aux->ev[1 + gi], gst));
                continue;
            }
        }
        if (kind == KIND_MM)
            CIL_TRY(launch_mm_named<T>(kv.first, c.scheme, (int)kv.second.size(), dS, dls[gi], state,
                                       (const T *)mms[gi].tab, (const T *)mms[gi].tab2, (const T *)mms[gi].cst,
                                       c.model, c.dt, pa, gst));
        else
            CIL_TRY(launch_persistent<T>(kv.first, quad, shape, (int)kv.second.size(), dS, dls[gi], state,
                                         (const T *)tabs[gi], c.model, c.dt, pa, gst));
        if (aux) CIL_HIP(hipEventRecord(aux->ev[1 + gi], gst));
    }
    if (aside) CIL_TRY((*aside)());
    if (aux)
        for (int gi = 0; gi < ng; ++gi) CIL_HIP(hipStreamWaitEvent(c.st, aux->ev[1 + gi], 0));
    HostResults h;
    CIL_TRY(fetch_results(c, B, dsteps, dres, dstat, mx ? mx->sw : nullptr, &h));
    for (size_t gi = 0; gi < groups.size(); ++gi)
        for (int b : groups[gi]->second) {
            c.steps[b] = h.steps[b];
            c.fres[b] = h.res[b];
            c.status[b] = h.stat[b];
            if (mixed[gi]) c.sw[b] = h.sw[b];
        }
    return CIL_OK;
}

// The mixed kernel's continuation as a launch of its own (mode 2) over FP32
// solves that its FP32-phase launch (mode 1) left at their floor: FP64 steps,
// or the refinement form with `refine`.  state64: same element layout as
// `state`.
int run_phase2(SimCtx &c, const std::map<int, std::vector<int>> &byn, std::vector<DevSolve> &hs, DevSolve *dS,
               FusedKind kind, float *state, double *state64, long long *sw, bool refine, long long *dsteps,
               double *dres, int *dstat)
{
    if (byn.empty()) return CIL_OK;
    const int B = (int)hs.size();
    std::vector<void *> tabs, tabs64;
    for (auto &kv : byn) {
        void *t, *t64 = nullptr;
        if (kind == KIND_MM) {
            MmTables mt;
            CIL_TRY(make_mm_tables<float>(c, kv.first, kv.second, hs, &mt));
            t = mt.tab;
        } else {
            CIL_TRY(make_tables<float>(c, kv.first, kv.second, hs, &t, kQuadShape[quad_shape(true, kv.first)].vform));
        }
        if (!refine) CIL_TRY(polish_tables(c, kv.first, kv.second, hs, kind, &t64));
        tabs.push_back(t);
        tabs64.push_back(t64);
    }
    CIL_HIP(hipMemcpyAsync(dS, hs.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, c.st));
    std::vector<long long> hsteps(c.steps.begin(), c.steps.end());
    CIL_HIP(hipMemcpyAsync(dsteps, hsteps.data(), sizeof(long long) * B, hipMemcpyHostToDevice, c.st));
    const PersistArgs pa{(long long)c.max_steps, c.tol, c.check, 0.0, dsteps, dres, dstat, g_wave_priority};
    size_t gi = 0;
    for (auto &kv : byn) {
        int *dl;
        CIL_TRY(c.cb->alloc((void **)&dl, sizeof(int) * kv.second.size()));
        CIL_HIP(hipMemcpyAsync(dl, kv.second.data(), sizeof(int) * kv.second.size(), hipMemcpyHostToDevice, c.st));
        CIL_TRY(launch_mixed_named(kind, kv.first, (int)kv.second.size(), dS, dl, state, state64,
                                   (const float *)tabs[gi], (const double *)tabs64[gi], c.model, c.dt, pa, pa, sw,
                                   refine, 2, c.st));
        ++gi;
    }
    HostResults h;
    CIL_TRY(fetch_results(c, B, dsteps, dres, dstat, nullptr, &h));
    for (auto &kv : byn)
        for (int b : kv.second) {
            c.steps[b] = h.steps[b];
            c.fres[b] = h.res[b];
            c.status[b] = h.stat[b];
        }
    return CIL_OK;
}

// Second-order fused solves, line variant (path FUSED_LINE; n = 32, and n = 64
// in FP32, where state and history fit the LDS of one workgroup), one launch
// per grid side, in order on the caller's stream.
bool sbdf2_fused_supported(int n, bool f32) { return n == 32 || (n == 64 && f32); }

template <typename T>
int run_fused_sbdf2(SimCtx &c, const std::map<int, std::vector<int>> &byn, std::vector<DevSolve> &hs, DevSolve *dS,
                    T *state, double floor_coef, long long *dsteps, double *dres, int *dstat)
{
    if (byn.empty()) return CIL_OK;
    const bool f32 = std::is_same<T, float>::value;
    std::vector<void *> tabE, tabB;
    for (auto &kv : byn) {
        void *te, *tb;
        CIL_TRY(make_tables<T>(c, kv.first, kv.second, hs, &te, false, c.dt));
        CIL_TRY(make_tables<T>(c, kv.first, kv.second, hs, &tb, false, 2.0 * c.dt / 3.0));
        tabE.push_back(te);
        tabB.push_back(tb);
    }
    const int B = (int)hs.size();
    CIL_HIP(hipMemcpyAsync(dS, hs.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, c.st));
    std::vector<long long> hsteps(c.steps.begin(), c.steps.end());
    CIL_HIP(hipMemcpyAsync(dsteps, hsteps.data(), sizeof(long long) * B, hipMemcpyHostToDevice, c.st));
    PersistArgs pa{(long long)c.max_steps, c.tol, c.check, floor_coef, dsteps, dres, dstat, 0.0};
    int gi = 0;
    for (auto &kv : byn) {
        const int n = kv.first, nl = (int)kv.second.size();
        int *dl;
        CIL_TRY(c.cb->alloc((void **)&dl, sizeof(int) * nl));
        CIL_HIP(hipMemcpyAsync(dl, kv.second.data(), sizeof(int) * nl, hipMemcpyHostToDevice, c.st));
        const T *te = (const T *)tabE[gi], *tb = (const T *)tabB[gi];
        ++gi;
        const char *name = n == 32 ? (f32 ? "k_fused_sbdf2_f32_n32" : "k_fused_sbdf2_f64_n32") : "k_fused_sbdf2_f32_n64";
        const ProfMark pm = prof_begin(name, c.st);
        if (n == 32)
            hipLaunchKernelGGL((k_fused_sbdf2<T, 32>), dim3(nl), dim3(64), 0, c.st, dS, dl, state, te, tb, c.model,
                               c.dt, pa);
        else if constexpr (std::is_same<T, float>::value) {
            if (n == 64)
                hipLaunchKernelGGL((k_fused_sbdf2<T, 64>), dim3(nl), dim3(128), 0, c.st, dS, dl, state, te, tb,
                                   c.model, c.dt, pa);
        }
        prof_end(pm, c.st);
        CIL_TRY(check_launch(name));
    }
    HostResults h;
    CIL_TRY(fetch_results(c, B, dsteps, dres, dstat, nullptr, &h));
    for (auto &kv : byn)
        for (int b : kv.second) {
            c.steps[b] = h.steps[b];
            c.fres[b] = h.res[b];
            c.status[b] = h.stat[b];
        }
    return CIL_OK;
}

// Launch order of a split group's tiles: workgroups go round the eight XCDs, and a
// solve's tiles all go to one of them, whose L2 then holds its field between the
// passes (64 solves of 128^2: 25.8 us a step, 34.6 in the solves' order).  Solves in order of falling cost, each to the XCD with the least.
template <typename T>
int upload_items(PlainGroup<T> &g, hipStream_t st)
{
    constexpr int X = 8;
    std::vector<SplitItem<T>> per[X];
    std::vector<const std::vector<SplitItem<T>> *> order;
    for (auto &t : g.tiles) order.push_back(&t);
    std::stable_sort(order.begin(), order.end(), [](auto *a, auto *b) { return a->size() > b->size(); });
    for (auto *t : order) {
        auto *x = std::min_element(per, per + X, [](auto &a, auto &b) { return a.size() < b.size(); });
        x->insert(x->end(), t->begin(), t->end());
    }
    size_t most = 0;
    for (auto &x : per) most = std::max(most, x.size());
    SplitItem<T> none{};
    none.b = -1;
    for (size_t k = 0; k < most; ++k)
        for (auto &x : per) g.items.push_back(k < x.size() ? x[k] : none);
    CIL_HIP(hipMemcpyAsync(g.ditems, g.items.data(), sizeof(SplitItem<T>) * g.items.size(), hipMemcpyHostToDevice, st));
    return CIL_OK;
}

// Plain solves: host-driven lockstep loop from a common step `start`; a
// launch per stage per step, the residual read back every check_every steps.
template <typename T>
int run_plain(SimCtx &c, std::vector<PlainGroup<T>> &groups, const DevSolve *dS, T *state, int64_t start,
              double floor_coef, StepResults R, int B)
{
    // the results as R holds them: residuals, maxima, flags (half a word each)
    std::vector<unsigned long long> stage(2 * (size_t)B + (B + 1) / 2);
    const size_t rbytes = (2 * sizeof(unsigned long long) + sizeof(int)) * (size_t)B;
    const unsigned long long *h_resid = stage.data(), *h_maxabs = h_resid + B;
    const int *h_bad = (const int *)(h_maxabs + B);
    int64_t step = start;
    auto any_active = [&]() {
        for (auto &g : groups)
            if (!g.active.empty()) return true;
        return false;
    };
    while (step < c.max_steps && any_active()) {
        const int64_t next = std::min<int64_t>(c.max_steps, (step / c.check + 1) * c.check);
        const int K = (int)(next - step);
        for (auto &g : groups) {
            if (g.active.empty()) continue;
            const int nl = (int)g.active.size();
            CIL_HIP(hipMemcpyAsync(g.dlist, g.active.data(), sizeof(int) * nl, hipMemcpyHostToDevice, c.st));
            hipLaunchKernelGGL(k_clear_results, dim3((nl + 255) / 256), dim3(256), 0, c.st, g.dlist, nl, R);
            if (g.split) {
                if (g.items.empty()) CIL_TRY(upload_items(g, c.st));
                constexpr bool f32 = std::is_same<T, float>::value;
                SplitArgs<T> a{};
                a.items = g.ditems;
                a.state = state;
                a.c0 = g.c0;
                a.ct = g.ct;
                a.res = R;
                const ProfMark pm = prof_begin(c.scheme ? (f32 ? "split_step_sbdf2_f32" : "split_step_sbdf2_f64")
                                                        : (f32 ? "split_step_f32" : "split_step_f64"), c.st);
                CIL_TRY(launch_split<T>(a, (int)g.items.size(), c.model, c.dt, K, c.scheme != 0, step == 0, c.st));
                prof_end(pm, c.st);
                continue;
            }
            const Sbdf2Args<T> bdf{(T *)c.uh, (T *)c.fh, step};
            CIL_TRY(launch_plain<T>(g, dS, state, nl, c.model, c.dt, K, R, c.st, c.scheme ? &bdf : nullptr));
        }
        CIL_HIP(hipMemcpyAsync(stage.data(), R.resid, rbytes, hipMemcpyDeviceToHost, c.st));
        CIL_TRY(stream_wait(c.st));
        step = next;
        for (auto &g : groups) {
            std::vector<int> keep;
            for (int b : g.active) {
                double dmax, amax;
                std::memcpy(&dmax, &h_resid[b], 8);
                std::memcpy(&amax, &h_maxabs[b], 8);
                const double r = dmax / c.dt;
                c.steps[b] = step;
                if (h_bad[b]) {
                    c.status[b] = CIL_SOLVE_NONFINITE;
                    c.fres[b] = NAN;
                    continue;
                }
                c.fres[b] = r;
                if (c.tol > 0.0 && r < c.tol) {
                    c.status[b] = CIL_SOLVE_OK;
                    continue;
                }
                if (c.tol > 0.0 && floor_coef > 0.0 && r < floor_coef * amax) {
                    c.status[b] = CIL_SOLVE_FP32_FLOOR;
                    continue;
                }
                if (step >= c.max_steps) {
                    c.status[b] = c.tol > 0.0 ? CIL_SOLVE_MAXSTEPS : CIL_SOLVE_OK;
                    continue;
                }
                keep.push_back(b);
            }
            if (g.split && keep.size() < g.active.size()) {
                g.items.clear();
                g.tiles.erase(std::remove_if(g.tiles.begin(), g.tiles.end(),
                                             [&](const std::vector<SplitItem<T>> &t) {
                                                 return std::find(keep.begin(), keep.end(), t[0].b) == keep.end();
                                             }),
                              g.tiles.end());
            }
            g.active.swap(keep);
        }
    }
    return CIL_OK;
}

// The solves of `byn` as one split group: tables per side, items per tile.
template <typename T>
int make_split_group(SimCtx &c, const std::map<int, std::vector<int>> &byn, std::vector<DevSolve> &hs, PlainGroup<T> *g)
{
    size_t work = 0, solves = 0;
    for (auto &kv : byn) {
        work += (size_t)2 * mm_padded(kv.first) * mm_padded(kv.first) * kv.second.size();
        solves += kv.second.size();
    }
    T *w, *h = nullptr;
    if (std::is_same<T, float>::value && c.model != CIL_FHN && c.model != CIL_HEAT) {    // (kOffset)
        CIL_TRY(c.cb->alloc((void **)&g->c0, sizeof(T) * 2 * solves));
        CIL_TRY(c.cb->alloc((void **)&g->ct, sizeof(T) * 32 * solves));
    }
    CIL_TRY(c.cb->alloc((void **)&w, sizeof(T) * work));
    if (c.scheme) CIL_TRY(c.cb->alloc((void **)&h, sizeof(T) * 2 * work));
    size_t most = 0;
    for (auto &kv : byn) {
        MmTables mt;
        CIL_TRY(make_mm_tables<T>(c, kv.first, kv.second, hs, &mt, c.scheme ? 2.0 * c.dt / 3.0 : 0.0));
        const int N = mm_padded(kv.first), per = 2 * N * 8;           // values to a tile
        for (int b : kv.second) {
            std::vector<SplitItem<T>> tiles(N / 8);
            for (int t = 0; t < N / 8; ++t) {
                const size_t div = (size_t)hs[b].tab * 2 * N * N + (size_t)t * per;
                tiles[t] = SplitItem<T>{hs[b], b, t, (int)g->tiles.size(), 0, (const T *)mt.cst, (const T *)mt.tab + div,
                                     c.scheme ? (const T *)mt.tab2 + div : nullptr, w,
                                     h ? h + (size_t)2 * t * per : nullptr, {}, {}};
                split_offsets(c.model, hs[b].p, tiles[t].u0, tiles[t].least);
            }
            g->tiles.push_back(std::move(tiles));
            g->active.push_back(b);
            w += (size_t)2 * N * N;
            if (h) h += (size_t)4 * N * N;
            most = std::max<size_t>(most, N / 8);
        }
    }
    g->split = true;
    // the fullest XCD exceeds the average by at most one solve
    size_t all = 0;
    for (auto &t : g->tiles) all += t.size();
    CIL_TRY(c.cb->alloc((void **)&g->ditems, sizeof(SplitItem<T>) * (all + 8 * most)));
    CIL_TRY(c.cb->alloc((void **)&g->dlist, sizeof(int) * g->active.size()));
    return CIL_OK;
}

template <typename T>
int make_plain_groups(SimCtx &c, const std::map<int, std::vector<int>> &byn, std::vector<DevSolve> &hs, bool split,
                      std::vector<PlainGroup<T>> &out)
{
    std::map<int, std::vector<int>> tiled;
    if (split)
        for (auto &kv : byn)
            if (split_supported(kv.first)) tiled.insert(kv);
    if (!tiled.empty()) {
        PlainGroup<T> g;
        CIL_TRY(make_split_group(c, tiled, hs, &g));
        out.push_back(std::move(g));
    }
    for (auto &kv : byn) {
        if (tiled.count(kv.first)) continue;
        PlainGroup<T> g;
        g.n = kv.first;
        g.active = kv.second;
        g.work_cap = kv.second.size();
        CIL_TRY(c.cb->alloc((void **)&g.dlist, sizeof(int) * g.work_cap));
        CIL_TRY(c.cb->alloc(&g.work, sizeof(T) * (size_t)2 * g.work_cap * 2 * g.n * g.n));
        out.push_back(g);
    }
    return CIL_OK;
}

}  // namespace

int simulate_impl(cil_model model, cil_precision prec, const cil_problem *probs, int B, void *state,
                  const int64_t *offs, const cil_stepping *stp, cil_solve_report *reports, hipStream_t st, int scheme)
{
    const bool f32 = (prec == CIL_FP32);
    const int floor_ulps = stp->fp32_floor_ulps > 0 ? stp->fp32_floor_ulps : 8;
    CallBuffers cb;
    SimCtx c;
    c.model = (int)model;
    c.dt = stp->dt;
    c.tol = stp->tol;
    c.max_steps = stp->max_steps;
    c.check = stp->check_every;
    c.floor_coef32 = (f32 && stp->tol > 0.0) ? floor_ulps * std::ldexp(1.0, -24) / stp->dt : 0.0;
    c.st = st;
    c.cb = &cb;
    c.steps.assign(B, 0);
    c.fres.assign(B, 0.0);
    c.status.assign(B, CIL_SOLVE_OK);
    const bool polish = f32 && stp->polish && stp->tol > 0.0;
    c.polish = polish ? stp->polish : 0;
    FusedKind kind = fused_kind(stp->path);
    if (scheme) {
        if (kind == KIND_QUAD) kind = KIND_MM;                // a quad code shape chosen by option: not this scheme's
        if (stp->path == CIL_PATH_FUSED_QUAD)
            return set_error(CIL_EUNSUPPORTED, "the second-order stepper has no quad-lane kernel");
        if (polish)
            return set_error(CIL_EUNSUPPORTED, "the second-order stepper has no FP64 polish: set polish = 0");
    }
    c.scheme = scheme;

    std::vector<DevSolve> hs(B);
    std::vector<int64_t> elems(B);
    int64_t total = 0;
    for (int b = 0; b < B; ++b) {
        const cil_problem &pr = probs[b];
        DevSolve d{};
        d.n = pr.n;
        d.off = offs ? offs[b] : total;
        const double h = pr.L / (double)(pr.n - 1);
        d.inv_h2 = 1.0 / (h * h);
        d.nu[0] = pr.nu[0];
        d.nu[1] = pr.nu[1];
        for (int k = 0; k < 4; ++k) d.p[k] = pr.p[k];
        hs[b] = d;
        elems[b] = 2ll * pr.n * pr.n;
        total += elems[b];
    }

    // phase 1: fused sides run persistently, the rest in the lockstep loop (sides
    // of 65 to 128 tile by tile on the matrix cores, others in plain kernels)
    const bool autop = stp->path == CIL_PATH_AUTO;
    std::map<int, std::vector<int>> fused_byn, plain_byn;
    int64_t waves = 0;
    for (const DevSolve &s : hs) waves += mm_padded(s.n) / 8;
    for (int b = 0; b < B; ++b) {
        const int n = hs[b].n;
        const bool fs = persistent_supported(n, f32, stp->path) &&
                        (!scheme || stp->path < CIL_PATH_FUSED || sbdf2_fused_supported(n, f32));
        if (stp->path >= CIL_PATH_FUSED && !fs)
            return set_error(CIL_EUNSUPPORTED, "no fused %sstepper for n = %d in %s", scheme ? "second-order " : "", n,
                             f32 ? "FP32" : "FP64");
        if (fs && !(autop && kind == KIND_MM && tile_by_tile(n, f32, waves, stp->check_every))) fused_byn[n].push_back(b);
        else plain_byn[n].push_back(b);
    }
    bool plain_hist = false;                         // the plain kernels keep the history in HBM
    for (auto &kv : plain_byn) plain_hist |= !(autop && split_supported(kv.first));
    if (scheme && plain_hist) {
        int64_t end = 0;
        for (int b = 0; b < B; ++b) end = std::max<int64_t>(end, hs[b].off + elems[b]);
        const size_t es = f32 ? sizeof(float) : sizeof(double);
        CIL_TRY(cb.alloc(&c.uh, es * (size_t)end));
        CIL_TRY(cb.alloc(&c.fh, es * (size_t)end));
    }
    DevSolve *dS;
    long long *dsteps;
    double *dres;
    int *dstat;
    CIL_TRY(cb.alloc((void **)&dS, sizeof(DevSolve) * B));
    CIL_TRY(cb.alloc((void **)&dsteps, sizeof(long long) * B));
    CIL_TRY(cb.alloc((void **)&dres, sizeof(double) * B));
    CIL_TRY(cb.alloc((void **)&dstat, sizeof(int) * B));
    CIL_TRY(fill_zero(dstat, sizeof(int) * B, st));
    StepResults R;
    CIL_TRY(cb.alloc((void **)&R.resid, (2 * sizeof(unsigned long long) + sizeof(int)) * B));   // read back as one block
    R.maxabs = R.resid + B;
    R.bad = (int *)(R.maxabs + B);

    c.sw.assign(B, -1);
    MixedArgs mx{nullptr, nullptr, c.polish == 2};
    bool use_mixed = false;
    if (polish)
        for (auto &kv : fused_byn) use_mixed |= mixed_supported(kv.first, kind);
    if (use_mixed) {
        int64_t end = 0;
        for (int b = 0; b < B; ++b) end = std::max<int64_t>(end, hs[b].off + elems[b]);
        CIL_TRY(cb.alloc((void **)&mx.state64, sizeof(double) * (size_t)end));
        CIL_TRY(cb.alloc((void **)&mx.sw, sizeof(long long) * B));
    }
    std::vector<PlainGroup<float>> pg32;
    std::vector<PlainGroup<double>> pg64;
    if (f32) CIL_TRY(make_plain_groups<float>(c, plain_byn, hs, autop, pg32));
    else CIL_TRY(make_plain_groups<double>(c, plain_byn, hs, autop, pg64));
    const std::function<int()> lockstep = [&]() -> int {
        return f32 ? run_plain<float>(c, pg32, dS, (float *)state, 0, c.floor_coef32, R, B)
                   : run_plain<double>(c, pg64, dS, (double *)state, 0, 0.0, R, B);
    };
    const std::function<int()> *aside = plain_byn.empty() ? nullptr : &lockstep;
    if (scheme && kind == KIND_LINE) {
        if (f32) CIL_TRY(run_fused_sbdf2<float>(c, fused_byn, hs, dS, (float *)state, c.floor_coef32, dsteps, dres, dstat));
        else CIL_TRY(run_fused_sbdf2<double>(c, fused_byn, hs, dS, (double *)state, 0.0, dsteps, dres, dstat));
    } else if (f32) {
        CIL_TRY(run_fused<float>(c, fused_byn, hs, dS, (float *)state, kind, c.floor_coef32, dsteps, dres, dstat,
                                 use_mixed ? &mx : nullptr, aside));
    } else {
        CIL_TRY(run_fused<double>(c, fused_byn, hs, dS, (double *)state, kind, 0.0, dsteps, dres, dstat, nullptr, aside));
    }
    if (fused_byn.empty() && aside) {
        CIL_HIP(hipMemcpyAsync(dS, hs.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, st));
        CIL_TRY(lockstep());
    }

    // phase 2: FP32 solves stopped at the FP32 floor continue: those whose
    // FP32 phase ran in the mixed kernel (separate polish) in its second
    // launch, the others in FP64 steps
    std::vector<int64_t> steps64(B, 0);
    std::vector<int> promoted;
    std::map<int, std::vector<int>> cont_byn;
    for (int b = 0; b < B; ++b) {
        if (c.sw[b] >= 0) steps64[b] = c.steps[b] - c.sw[b];     // polished inside the mixed launch
        if (!polish || c.status[b] != CIL_SOLVE_FP32_FLOOR) continue;
        if (c.sw[b] >= 0) cont_byn[hs[b].n].push_back(b);
        else promoted.push_back(b);
    }
    if (!cont_byn.empty()) {
        for (auto &kv : cont_byn)
            for (int b : kv.second) c.status[b] = CIL_SOLVE_OK;
        CIL_TRY(run_phase2(c, cont_byn, hs, dS, kind, (float *)state, mx.state64, mx.sw, c.polish == 2, dsteps, dres,
                           dstat));
        for (auto &kv : cont_byn)
            for (int b : kv.second) steps64[b] = c.steps[b] - c.sw[b];
    }
    if (!promoted.empty()) {
        std::vector<DevSolve> hs64 = hs;
        int64_t t = 0;
        for (int b = 0; b < B; ++b) {
            hs64[b].off = t;
            t += elems[b];
        }
        double *state64;
        DevSolve *dS64;
        int *dprom;
        CIL_TRY(cb.alloc((void **)&state64, sizeof(double) * std::max<int64_t>(t, 1)));
        CIL_TRY(cb.alloc((void **)&dS64, sizeof(DevSolve) * B));
        CIL_TRY(cb.alloc((void **)&dprom, sizeof(int) * promoted.size()));
        CIL_HIP(hipMemcpyAsync(dS, hs.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, st));
        CIL_HIP(hipMemcpyAsync(dS64, hs64.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, st));
        CIL_HIP(hipMemcpyAsync(dprom, promoted.data(), sizeof(int) * promoted.size(), hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL((k_convert_solves<float, double>), dim3(16, (unsigned)promoted.size()), dim3(256), 0, st,
                           (const DevSolve *)dS, (const DevSolve *)dS64, dprom, (const float *)state, state64);
        CIL_TRY(check_launch("k_convert_solves"));
        std::vector<int64_t> before(B);
        for (int b = 0; b < B; ++b) before[b] = c.steps[b];
        std::map<int, std::vector<int>> fz;                            // n -> solves (fused FP64)
        std::map<std::pair<int, int64_t>, std::vector<int>> pz;        // (n, start) -> solves (plain FP64)
        for (int b : promoted) {
            c.status[b] = CIL_SOLVE_OK;
            if (persistent_supported(hs[b].n, false, stp->path)) fz[hs[b].n].push_back(b);
            else pz[std::make_pair(hs[b].n, c.steps[b])].push_back(b);
        }
        CIL_TRY(run_fused<double>(c, fz, hs64, dS64, state64, kind, 0.0, dsteps, dres, dstat));
        for (auto &kv : pz) {
            std::map<int, std::vector<int>> one;
            one[kv.first.first] = kv.second;
            std::vector<PlainGroup<double>> pg;
            CIL_TRY(make_plain_groups<double>(c, one, hs64, autop, pg));
            CIL_HIP(hipMemcpyAsync(dS64, hs64.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, st));
            CIL_TRY(run_plain<double>(c, pg, dS64, state64, kv.first.second, 0.0, R, B));
        }
        for (int b : promoted) steps64[b] = c.steps[b] - before[b];
        hipLaunchKernelGGL((k_convert_solves<double, float>), dim3(16, (unsigned)promoted.size()), dim3(256), 0, st,
                           (const DevSolve *)dS64, (const DevSolve *)dS, dprom, (const double *)state64, (float *)state);
        CIL_TRY(check_launch("k_convert_solves"));
    }
    CIL_TRY(stream_wait(st));
    cb.done = true;

    int rc = CIL_OK;
    for (int b = 0; b < B; ++b) {
        if (c.status[b] == CIL_SOLVE_NONFINITE) rc = CIL_ENONFINITE;
        if (reports) {
            reports[b].steps_taken = c.steps[b];
            reports[b].steps_fp64 = f32 ? steps64[b] : 0;
            reports[b].final_resid = c.fres[b];
            reports[b].status = c.status[b];
            reports[b].reserved = 0;
        }
    }
    if (rc == CIL_ENONFINITE) set_error(rc, "a solve produced a non-finite value");
    return rc;
}

// ------------------------------------------------------------------ plans
// A simulate plan binds one batch of fused solves (problems, layout,
// stepping, the state buffer) to device-resident spectral tables, solve
// descriptors and per-solve result arrays, and to one instantiated HIP graph:
// a clear of the results, then one persistent kernel per grid side, forked
// over plan-owned streams (default priority) and joined.  Each launch replays
// the graph: every solve starts at step 0 from what the state holds.
struct SimPlan {
    struct Group {
        int n = 0;
        std::vector<int> ids;
        int shape = 0;
        void *tab[2] = {nullptr, nullptr};    // X-form, V-form divisor tables (line and quad kernels)
        MmTables mm;                          // matrix-core kernel's
        bool use_mm = false;
        int *dl = nullptr;
        double tuned_ms[kQuadShapes] = {}, mm_ms = 0.0;
    };
    int dev = 0;
    int model = 0;
    bool f32 = false, quad = true, mm = false;    // mm: groups run on the matrix cores unless tuning finds a faster shape
    double dt = 0.0;
    PersistArgs pa{};
    void *state = nullptr;
    size_t state_bytes = 0;
    int B = 0;
    std::vector<DevSolve> hs;
    std::vector<Group> groups;            // launch order: most expensive first
    CallBuffers bufs;
    DevSolve *dS = nullptr;
    std::vector<hipStream_t> st;          // st[0] captures; st[g] runs group g
    std::vector<hipEvent_t> ev;           // ev[0] fork, ev[g] join of group g
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    ~SimPlan()
    {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        for (hipStream_t s : st) (void)hipStreamDestroy(s);
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    }
};

namespace {

// tables of group g for the divisor form of `shape` (built once per form)
int plan_tables(SimPlan &p, SimPlan::Group &g, int shape, hipStream_t st)
{
    const int vf = (p.quad && kQuadShape[shape].vform) ? 1 : 0;
    if (g.tab[vf]) return CIL_OK;
    SimCtx c;
    c.model = p.model;
    c.dt = p.dt;
    c.st = st;
    c.cb = &p.bufs;
    if (p.f32) CIL_TRY(make_tables<float>(c, g.n, g.ids, p.hs, &g.tab[vf], vf != 0));
    else CIL_TRY(make_tables<double>(c, g.n, g.ids, p.hs, &g.tab[vf], vf != 0));
    // the table index of each solve depends only on (h, nu) order within the
    // group, the same for both forms; descriptors are re-sent after a build
    CIL_HIP(hipMemcpyAsync(p.dS, p.hs.data(), sizeof(DevSolve) * p.B, hipMemcpyHostToDevice, st));
    return CIL_OK;
}

int plan_mm_tables(SimPlan &p, SimPlan::Group &g, hipStream_t st)
{
    SimCtx c;
    c.model = p.model;
    c.dt = p.dt;
    c.st = st;
    c.cb = &p.bufs;
    if (p.f32) CIL_TRY(make_mm_tables<float>(c, g.n, g.ids, p.hs, &g.mm));
    else CIL_TRY(make_mm_tables<double>(c, g.n, g.ids, p.hs, &g.mm));
    CIL_HIP(hipMemcpyAsync(p.dS, p.hs.data(), sizeof(DevSolve) * p.B, hipMemcpyHostToDevice, st));
    return CIL_OK;
}

// shape < 0: the matrix-core kernel
int plan_launch_group(SimPlan &p, SimPlan::Group &g, int shape, void *state, const PersistArgs &pa, hipStream_t st)
{
    if (shape < 0) {
        if (p.f32)
            return launch_mm_named<float>(g.n, 0, (int)g.ids.size(), p.dS, g.dl, (float *)state, (const float *)g.mm.tab,
                                          nullptr, (const float *)g.mm.cst, p.model, p.dt, pa, st);
        return launch_mm_named<double>(g.n, 0, (int)g.ids.size(), p.dS, g.dl, (double *)state,
                                       (const double *)g.mm.tab, nullptr, (const double *)g.mm.cst, p.model, p.dt, pa,
                                       st);
    }
    const int vf = (p.quad && kQuadShape[shape].vform) ? 1 : 0;
    if (p.f32)
        return launch_persistent<float>(g.n, p.quad, shape, (int)g.ids.size(), p.dS, g.dl, (float *)state,
                                        (const float *)g.tab[vf], p.model, p.dt, pa, st);
    return launch_persistent<double>(g.n, p.quad, shape, (int)g.ids.size(), p.dS, g.dl, (double *)state,
                                     (const double *)g.tab[vf], p.model, p.dt, pa, st);
}

// the graph's work, enqueued on the capturing stream p.st[0]
int plan_enqueue(SimPlan &p)
{
    hipStream_t cs = p.st[0];
    CIL_TRY(fill_zero(p.pa.steps, sizeof(long long) * p.B, cs));
    CIL_TRY(fill_zero(p.pa.resid, sizeof(double) * p.B, cs));
    CIL_TRY(fill_zero(p.pa.status, sizeof(int) * p.B, cs));
    const int ng = (int)p.groups.size();
    if (ng > 1) CIL_HIP(hipEventRecord(p.ev[0], cs));
    for (int g = 1; g < ng; ++g) CIL_HIP(hipStreamWaitEvent(p.st[g], p.ev[0], 0));
    for (int g = 0; g < ng; ++g) {
        SimPlan::Group &gr = p.groups[g];
        CIL_TRY(plan_launch_group(p, gr, gr.use_mm ? -1 : gr.shape, p.state, p.pa, p.st[g]));
    }
    for (int g = 1; g < ng; ++g) {
        CIL_HIP(hipEventRecord(p.ev[g], p.st[g]));
        CIL_HIP(hipStreamWaitEvent(cs, p.ev[g], 0));
    }
    return CIL_OK;
}

int plan_build_graph(SimPlan &p)
{
    if (p.exec) (void)hipGraphExecDestroy(p.exec);
    if (p.graph) (void)hipGraphDestroy(p.graph);
    p.exec = nullptr;
    p.graph = nullptr;
    CIL_HIP(hipStreamBeginCapture(p.st[0], hipStreamCaptureModeThreadLocal));
    const int rc = plan_enqueue(p);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(p.st[0], &g);
    if (rc != CIL_OK) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
    }
    if (e != hipSuccess) return set_error(CIL_EDEVICE, "graph capture failed: %s", hipGetErrorString(e));
    p.graph = g;
    CIL_HIP(hipGraphInstantiate(&p.exec, g, nullptr, nullptr, 0));
    return CIL_OK;
}

}  // namespace

int plan_create(cil_model model, cil_precision prec, const cil_problem *probs, int B, void *state, const int64_t *offs,
                const cil_stepping *stp, hipStream_t st, SimPlan **out)
{
    const bool f32 = (prec == CIL_FP32);
    if (stp->path == CIL_PATH_PLAIN) return set_error(CIL_EUNSUPPORTED, "plans run the fused steppers only");
    if (f32 && stp->polish && stp->tol > 0.0)
        return set_error(CIL_EINVAL, "plans do not polish in FP64: set polish = 0 (FP32 floor is then a status)");
    std::unique_ptr<SimPlan> p(new SimPlan());
    CIL_TRY(current_device(&p->dev));
    p->model = (int)model;
    p->f32 = f32;
    const FusedKind kind = fused_kind(stp->path);
    p->quad = kind != KIND_LINE;
    p->mm = kind == KIND_MM;
    p->dt = stp->dt;
    p->state = state;
    p->B = B;
    p->hs.resize(B);
    int64_t total = 0, end = 0;
    std::map<int, std::vector<int>> byn;
    for (int b = 0; b < B; ++b) {
        const cil_problem &pr = probs[b];
        if (!fused_supported(pr.n, f32))
            return set_error(CIL_EUNSUPPORTED, "no fused stepper for n = %d in %s", pr.n, f32 ? "FP32" : "FP64");
        DevSolve d{};
        d.n = pr.n;
        d.off = offs ? offs[b] : total;
        const double h = pr.L / (double)(pr.n - 1);
        d.inv_h2 = 1.0 / (h * h);
        d.nu[0] = pr.nu[0];
        d.nu[1] = pr.nu[1];
        for (int k = 0; k < 4; ++k) d.p[k] = pr.p[k];
        p->hs[b] = d;
        total += 2ll * pr.n * pr.n;
        end = std::max<int64_t>(end, d.off + 2ll * pr.n * pr.n);
        byn[pr.n].push_back(b);
    }
    p->state_bytes = (size_t)end * (f32 ? 4 : 8);
    std::vector<std::pair<double, int>> order;
    for (auto &kv : byn) order.push_back({-(double)kv.first * kv.first * std::log2((double)kv.first) * kv.second.size(),
                                          kv.first});
    std::sort(order.begin(), order.end());
    CIL_TRY(p->bufs.alloc((void **)&p->dS, sizeof(DevSolve) * B));
    long long *dsteps;
    double *dres;
    int *dstat;
    CIL_TRY(p->bufs.alloc((void **)&dsteps, sizeof(long long) * B));
    CIL_TRY(p->bufs.alloc((void **)&dres, sizeof(double) * B));
    CIL_TRY(p->bufs.alloc((void **)&dstat, sizeof(int) * B));
    const double floor_coef =
        (f32 && stp->tol > 0.0) ? (stp->fp32_floor_ulps > 0 ? stp->fp32_floor_ulps : 8) * std::ldexp(1.0, -24) / stp->dt
                                : 0.0;
    p->pa = PersistArgs{(long long)stp->max_steps, stp->tol, stp->check_every, floor_coef, dsteps, dres, dstat,
                        g_wave_priority};
    CIL_HIP(hipMemcpyAsync(p->dS, p->hs.data(), sizeof(DevSolve) * B, hipMemcpyHostToDevice, st));
    for (auto &o : order) {
        SimPlan::Group g;
        g.n = o.second;
        g.ids = byn[g.n];
        g.shape = p->quad ? quad_shape(f32, g.n) : 0;
        g.use_mm = p->mm;
        CIL_TRY(p->bufs.alloc((void **)&g.dl, sizeof(int) * g.ids.size()));
        CIL_HIP(hipMemcpyAsync(g.dl, g.ids.data(), sizeof(int) * g.ids.size(), hipMemcpyHostToDevice, st));
        p->groups.push_back(g);
    }
    for (auto &g : p->groups) CIL_TRY(p->mm ? plan_mm_tables(*p, g, st) : plan_tables(*p, g, g.shape, st));
    const int ng = (int)p->groups.size();
    for (int g = 0; g < std::max(ng, 1); ++g) {
        hipStream_t s;
        CIL_HIP(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
        p->st.push_back(s);
        hipEvent_t e;
        CIL_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        p->ev.push_back(e);
    }
    CIL_HIP(hipStreamSynchronize(st));     // uploads done before capture and before host vectors go
    CIL_TRY(plan_build_graph(*p));
    *out = p.release();
    return CIL_OK;
}

int plan_tune(SimPlan *p, int64_t steps, hipStream_t st)
{
    if (!p->quad) return set_error(CIL_EINVAL, "tuning chooses among the quad-lane shapes (path is FUSED_LINE)");
    if (steps < 0) return set_error(CIL_EINVAL, "tuning needs steps >= 0");
    CIL_HIP(hipSetDevice(p->dev));
    CallBuffers tb;
    void *scratch;
    long long *tsteps;
    double *tres;
    int *tstat;
    CIL_TRY(tb.alloc(&scratch, p->state_bytes));
    CIL_TRY(tb.alloc((void **)&tsteps, sizeof(long long) * p->B));
    CIL_TRY(tb.alloc((void **)&tres, sizeof(double) * p->B));
    CIL_TRY(tb.alloc((void **)&tstat, sizeof(int) * p->B));
    // steps > 0: fixed-length trials (no stop rule); 0: the plan's own stepping
    const PersistArgs pa = steps > 0 ? PersistArgs{(long long)steps, 0.0, (int)std::min<int64_t>(steps, 1 << 30), 0.0,
                                                   tsteps, tres, tstat}
                                     : PersistArgs{p->pa.max_steps, p->pa.tol, p->pa.check, p->pa.floor_coef, tsteps,
                                                   tres, tstat, p->pa.prio};
    hipEvent_t a, b;
    CIL_HIP(hipEventCreate(&a));
    CIL_HIP(hipEventCreate(&b));
    int rc = CIL_OK;
    for (auto &g : p->groups) {
        // the quad-lane shapes, then (shape -1) the matrix-core kernel where the plan's path includes it
        int best = -1;
        for (int s = 0; s <= kQuadShapes && rc == CIL_OK; ++s) {
            const bool mm = s == kQuadShapes;
            if (mm && !p->mm) break;
            if (!mm) rc = plan_tables(*p, g, s, st);
            float ms = 0.0f;
            for (int rep = 0; rep < 2 && rc == CIL_OK; ++rep) {
                // every trial starts from the same states (a copy of the bound state)
                if (hipMemcpyAsync(scratch, p->state, p->state_bytes, hipMemcpyDeviceToDevice, st) != hipSuccess ||
                    (rc = fill_zero(tsteps, sizeof(long long) * p->B, st)) != CIL_OK ||
                    hipEventRecord(a, st) != hipSuccess) {
                    if (rc == CIL_OK) rc = set_error(CIL_EDEVICE, "tuning copy failed");
                    break;
                }
                rc = plan_launch_group(*p, g, mm ? -1 : s, scratch, pa, st);
                if (rc == CIL_OK && (hipEventRecord(b, st) != hipSuccess || hipEventSynchronize(b) != hipSuccess ||
                                     hipEventElapsedTime(&ms, a, b) != hipSuccess))
                    rc = set_error(CIL_EDEVICE, "tuning timing failed");
            }
            if (rc != CIL_OK) break;
            if (mm) {
                g.mm_ms = ms;
                g.use_mm = ms <= g.tuned_ms[best];
                break;
            }
            g.tuned_ms[s] = ms;
            if (best < 0 || ms < g.tuned_ms[best]) best = s;
        }
        if (rc != CIL_OK) break;
        g.shape = best;
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    CIL_TRY(rc);
    CIL_HIP(hipStreamSynchronize(st));
    tb.done = true;
    return plan_build_graph(*p);
}

int plan_launch(SimPlan *p, hipStream_t st)
{
    const ProfMark pm = prof_begin("sim_plan_graph", st);
    CIL_HIP(hipGraphLaunch(p->exec, st));
    prof_end(pm, st);
    return CIL_OK;
}

int plan_report(SimPlan *p, cil_solve_report *reports, hipStream_t st)
{
    const int B = p->B;
    std::vector<long long> hsteps(B);
    std::vector<double> hres(B);
    std::vector<int> hstat(B);
    CIL_HIP(hipMemcpyAsync(hsteps.data(), p->pa.steps, sizeof(long long) * B, hipMemcpyDeviceToHost, st));
    CIL_HIP(hipMemcpyAsync(hres.data(), p->pa.resid, sizeof(double) * B, hipMemcpyDeviceToHost, st));
    CIL_HIP(hipMemcpyAsync(hstat.data(), p->pa.status, sizeof(int) * B, hipMemcpyDeviceToHost, st));
    CIL_HIP(hipStreamSynchronize(st));
    int rc = CIL_OK;
    for (int b = 0; b < B; ++b) {
        if (hstat[b] == CIL_SOLVE_NONFINITE) rc = CIL_ENONFINITE;
        if (reports) reports[b] = cil_solve_report{hsteps[b], 0, hres[b], hstat[b], 0};
    }
    if (rc == CIL_ENONFINITE) set_error(rc, "a solve produced a non-finite value");
    return rc;
}

int plan_groups(const SimPlan *p) { return (int)p->groups.size(); }

int plan_group_info(const SimPlan *p, int g, int *n, int *count, int *shape, double *tuned_ms)
{
    if (g < 0 || g >= (int)p->groups.size()) return set_error(CIL_EINVAL, "group %d out of range", g);
    const SimPlan::Group &G = p->groups[g];
    if (n) *n = G.n;
    if (count) *count = (int)G.ids.size();
    if (shape) *shape = G.shape;
    if (tuned_ms)
        for (int s = 0; s < kQuadShapes; ++s) tuned_ms[s] = G.tuned_ms[s];
    return CIL_OK;
}

int plan_group_kernel(const SimPlan *p, int g, int *kernel, double *matrix_ms)
{
    if (g < 0 || g >= (int)p->groups.size()) return set_error(CIL_EINVAL, "group %d out of range", g);
    const SimPlan::Group &G = p->groups[g];
    if (kernel) *kernel = G.use_mm ? CIL_KERNEL_MATRIX : p->quad ? CIL_KERNEL_QUAD : CIL_KERNEL_LINE;
    if (matrix_ms) *matrix_ms = G.mm_ms;
    return CIL_OK;
}

void plan_destroy(SimPlan *p)
{
    if (!p) return;
    (void)hipSetDevice(p->dev);
    (void)hipDeviceSynchronize();
    p->bufs.done = true;
    delete p;
}

}  // namespace cil
