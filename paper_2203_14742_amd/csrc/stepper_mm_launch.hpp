// Host launches and table builders of the matrix-core stepper, instantiated
// per precision by stepper_mm_f32.hip and stepper_mm_f64.hip.
#pragma once

#include "stepper_mm.hpp"

namespace cil {

// Spectral divisors in the column pass's register order,
// tab[t][tile][hb][lane][i] = w_kx w_ky / (1 + dt nu (lam_kx + lam_ky) / h^2)
// (w_0 = 1/n, w_k = 2/n: the inverse transforms' weights), 0 for padding.
template <typename T, typename Line>
__global__ void k_mm_tables(const TabSpec *specs, int ntab, int n, double dt, T *out)
{
    constexpr int N = Line::N, NS = Line::NS;
    const int t = blockIdx.y, e = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntab || e >= 2 * N * N) return;
    const int i = e & 3, lane = (e >> 2) & 63, hb = (e >> 8) % NS, tile = (e >> 8) / NS;
    const int sp = (lane >> 3) & 1, slot = 8 * tile + (lane & 7);
    const int kx = slot_mode<Line>(slot >> 4, slot & 15, n), ky = slot_mode<Line>(hb, 4 * (lane >> 4) + i, n);
    double v = 0.0;
    if (kx >= 0 && ky >= 0) {
        const TabSpec ts = specs[t];
        const double sx = sinpi((double)kx / (2.0 * n)), sy = sinpi((double)ky / (2.0 * n));
        const double lam = 4.0 * (sx * sx + sy * sy) * ts.inv_h2;
        const double w = (kx ? 2.0 : 1.0) * (ky ? 2.0 : 1.0);
        v = w / ((double)n * n * (1.0 + dt * (sp ? ts.nu1 : ts.nu0) * lam));
    }
    out[(size_t)t * 2 * N * N + e] = T(v);
}

// Constant blocks of LineDense for side n: cosines of the even modes (rows
// modes, columns positions), their transpose, the odd modes (symmetric).
template <typename T, int NB>
__global__ void k_mm_dense_const(int n, T *out)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 3 * NB * NB * 256) return;
    const int i = e & 3, lane = (e >> 2) & 63, k = e >> 8;
    const int bi = k % NB, bo = (k / NB) % NB, m = k / (NB * NB);
    const int r = 16 * bo + mma_row_label<T>(lane & 15), q = 16 * bi + 4 * (lane >> 4) + i;
    double v = 0.0;
    if (m == 2) {
        if (r < n / 2 && q < n / 2) v = cospi((double)((2 * r + 1) * (2 * q + 1)) / (2.0 * n));
    } else {
        const int mode = m == 0 ? r : q, pos = m == 0 ? q : r;
        if (2 * mode < n && pos < (n + 1) / 2) v = cospi((double)(mode * (2 * pos + 1)) / (double)n);
    }
    out[e] = T(v);
}

// The line of side n <= 128: f(LineType).
template <typename T, typename F>
int mm_line(int n, F &&f)
{
    if (n == 32) return f(Line32<T>{});
    if (n == 64) return f(Line64<T>{});
    if (n == 128) return f(Line128<T>{});
    if (n < 2) return CIL_EUNSUPPORTED;
    switch (mm_padded(n)) {
    case 32: return f(LineDense<T, 1>{});
    case 64: return f(LineDense<T, 2>{});
    case 96: return f(LineDense<T, 3>{});
    case 128: return f(LineDense<T, 4>{});
    default: return CIL_EUNSUPPORTED;
    }
}

// The line of side n and its launch shape: f(LineType, TPW, WPE), TPW the tiles
// per wavefront, WPE the wavefronts per SIMD to allocate registers for.
template <typename Line, int TPW, int WPE, typename F>
int mm_call(F &&f)
{
    return f(Line{}, std::integral_constant<int, TPW>{}, std::integral_constant<int, WPE>{});
}
// The second-order scheme keeps the history in registers too, which costs its
// FP32 64^2 and FP64 32^2 kernels one step of occupancy.
template <typename T, int SCHEME = 0, typename F>
int mm_dispatch(int n, F &&f)
{
    constexpr bool f32 = sizeof(T) == 4;
    constexpr int w32 = SCHEME && !f32 ? 3 : 4, w64 = SCHEME || !f32 ? 2 : 4;
    if (n == 32) return mm_call<Line32<T>, 1, w32>(f);
    if (n == 64) return mm_call<Line64<T>, 1, w64>(f);
    if (n < 2 || n > mm_max_side(f32)) return CIL_EUNSUPPORTED;
    if constexpr (f32) {
        if (n == 128) return mm_call<Line128<T>, 2, 2>(f);
        if (mm_padded(n) == 128) return mm_call<LineDense<T, 4>, 2, 2>(f);
    }
    // (40000 FP64 solves of side 4, a pass of 100 steps: 17.9 ms with all four tiles, 9.6 with
    // the two that hold lines; 10.9 by a kernel per stage)
    if (n <= 16) return mm_call<LineShort<T>, 1, w32>(f);
    switch (mm_padded(n)) {
    case 32: return mm_call<LineDense<T, 1>, 1, w32>(f);
    case 64: return mm_call<LineDense<T, 2>, 1, w64>(f);
    case 96: return mm_call<LineDense<T, 3>, 1, 3>(f);
    default: return CIL_EUNSUPPORTED;
    }
}

template <typename T>
int mm_make_tables(int n, const TabSpec *specs, int ntab, double dt, T *out, hipStream_t st)
{
    return mm_line<T>(n, [&](auto line) -> int {
        using Line = decltype(line);
        hipLaunchKernelGGL((k_mm_tables<T, Line>), dim3((2 * Line::N * Line::N + 255) / 256, ntab), dim3(256), 0, st,
                           specs, ntab, n, dt, out);
        return check_launch("k_mm_tables");
    });
}

template <typename T>
int mm_make_consts(int n, T *out, hipStream_t st)
{
    return mm_line<T>(n, [&](auto line) -> int {
        using Line = decltype(line);
        if constexpr (Line::kRagged) {
            constexpr int NB = Line::N / 32;
            hipLaunchKernelGGL((k_mm_dense_const<T, NB>), dim3(3 * NB * NB), dim3(256), 0, st, n, out);
            return check_launch("k_mm_dense_const");
        } else {
            return CIL_OK;
        }
    });
}

template <typename T>
int launch_mm(int n, int scheme, int nl, const DevSolve *S, const int *list, T *state, const T *tab, const T *tab2,
              const T *cst, int model, double dt, const PersistArgs &pa, hipStream_t st)
{
    auto go = [&](auto line, auto tpw, auto wpe, auto sch) -> int {
        using Line = decltype(line);
        launch_mm_line<T, Line, decltype(sch)::value, decltype(tpw)::value, decltype(wpe)::value>(
            nl, S, list, state, tab, tab2, cst, model, dt, pa, st);
        return CIL_OK;
    };
    using std::integral_constant;
    if (scheme)
        return mm_dispatch<T, 1>(n, [&](auto l, auto t, auto w) { return go(l, t, w, integral_constant<int, 1>{}); });
    return mm_dispatch<T, 0>(n, [&](auto l, auto t, auto w) { return go(l, t, w, integral_constant<int, 0>{}); });
}

}  // namespace cil
