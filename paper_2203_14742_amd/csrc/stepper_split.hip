// The matrix-core stepper over many compute units: a wavefront per tile of
// eight grid lines, a launch per pass; sides 65 .. 128.
//
// The persistent kernel (stepper_mm.hpp) keeps a solve on one compute unit,
// which holds an FP64 field of side 96 at most and has four matrix cores of
// the chip's 1024.  Here a step is two launches over the tiles of all solves
// of the call, whatever their sides, with the field between them in memory:
//   row pass     row inverse, explicit reaction, row forward (and, where asked,
//                the state written and the stop rule's residual taken);
//   column pass  column forward, spectral divide, column inverse, in place.
// The passes are the persistent kernel's, on the same tiles (lanes l and l ^ 8
// hold the two species at the same points) and the same transforms.
//
// What bounds it: at few solves the latency of a launch and of its loads, then
// the matrix cores (a pass of a 128^2 solve is 64 products of 27 ns for each
// of 16 wavefronts, of any other side over 96 256 of them).  FHN 128^2, us per
// step, against a kernel per stage with one output value per lane: 1 solve
// 12.6 / 35.8, 8 13.0 / 109, 64 25.8 / 756, 256 66.5 / 2970; 112^2: 1 solve 23.4 /
// 35.1, 64 36.4 / 524.
#include "stepper_mm.hpp"

namespace cil {

namespace {

// f(Line) for a side of 65 .. 128
template <typename T, typename F>
__host__ __device__ __forceinline__ void split_dispatch(int n, F &&f)
{
    if (n == 128) f(Line128<T>{});
    else if (n > 96) f(LineDense<T, 4>{});
    else f(LineDense<T, 3>{});
}

template <int MODEL, typename T, typename Line>
__device__ __forceinline__ void row_pass(const SplitArgs<T> &a, const SplitItem<T> &it)
{
    using V = Vec4<T>;
    constexpr int N = Line::N, NS = Line::NS, ROR8 = 0x128;
    constexpr bool RAG = Line::kRagged;
    const int lane = threadIdx.x, c = lane & 15, sp = c >> 3, g4 = 4 * (lane >> 4);
    const DevSolve &s = it.s;
    const int line = 8 * it.tile + (c & 7), n = RAG ? s.n : N;
    Line L;
    L.init(it.cst, lane);
    T *const row = it.work + ((size_t)sp * N + line) * N + g4;
    const auto ub = make_rsrc(a.state + s.off, 2u * n * n * sizeof(T));
    const int rn = slot_pos<Line>(line >> 4, line & 15, n);
    const bool rok = slot_valid<Line>(line >> 4, line & 15, n);
    // byte offset of slot (hb, i) in the solve's state; padding reads 0 and is not written
    auto real = [&](int hb, int i) __attribute__((always_inline)) { return rok && slot_valid<Line>(hb, g4 + i, n); };
    auto at = [&](int hb, int i) __attribute__((always_inline)) {
        const unsigned e = (unsigned)((sp * n + rn) * n + slot_pos<Line>(hb, g4 + i, n)) * (unsigned)sizeof(T);
        return !RAG || real(hb, i) ? e : 0xFFFFFF00u;
    };
    // FP32 transforms act on u - u* (steady_value); FP64 ones on u
    T c0 = T(0);
    if constexpr (kOffset<MODEL, T>) c0 = a.c0[2 * it.k + sp];
    V x[NS], X[NS];
    if (a.flags & SPLIT_LOAD) {
#pragma unroll
        for (int hb = 0; hb < NS; ++hb)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[hb][i] = buf_load<T>(ub, at(hb, i), 0);
    } else {
#pragma unroll
        for (int hb = 0; hb < NS; ++hb) X[hb] = mm_load(row + hb * 16);
        L.inv(X, x);
        if constexpr (kOffset<MODEL, T>) {
#pragma unroll
            for (int hb = 0; hb < NS; ++hb) x[hb] += V(c0);
        }
    }
    if (a.flags & SPLIT_CHECK) {
        double d = 0.0, m = 0.0;
        int bad = 0;
#pragma unroll
        for (int hb = 0; hb < NS; ++hb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double v = (double)x[hb][i], dd = fabs(v - (double)buf_load<T>(ub, at(hb, i), 0));
                if (!RAG || real(hb, i)) {
                    bad |= !isfinite(v);
                    d = fmax(d, isnan(dd) ? 0.0 : dd);
                    m = fmax(m, isnan(v) ? 0.0 : fabs(v));
                }
            }
        d = wave_max(d);
        m = wave_max(m);
        bad = wave_or(bad);
        if (lane == 0) {
            atomicMax(&a.res.resid[it.b], (unsigned long long)__double_as_longlong(d));
            atomicMax(&a.res.maxabs[it.b], (unsigned long long)__double_as_longlong(m));
            if (bad) atomicOr(&a.res.bad[it.b], 1);
        }
    }
    if (a.flags & SPLIT_STORE) {
#pragma unroll
        for (int hb = 0; hb < NS; ++hb)
#pragma unroll
            for (int i = 0; i < 4; ++i) buf_store<T>((T)x[hb][i], ub, at(hb, i), 0);
    }
    if (!(a.flags & SPLIT_NEXT)) return;
    OwnReaction<MODEL, T> react;
    react.init(s.p, sp);
    if constexpr (kOffset<MODEL, T>) {                        // the tile's own choice, for the column pass
        const StepOffset<MODEL> offset{sp ? it.u0[1] : it.u0[0], sp ? it.least[1] : it.least[0]};
        const unsigned has = offset.template species<NS>(rok, [&](int hb, int i) __attribute__((always_inline)) {
            return slot_full<Line>(hb) || real(hb, i) ? fabsf(x[hb][i]) : __builtin_inff();
        });
        c0 = (has >> sp) & 1u ? offset.u0 : 0.0f;
        if ((lane & ~8) == 0) a.ct[(2 * it.k + sp) * 16 + it.tile] = c0;
    }
    const T cp = a.first ? T(0) : c0;                         // (no history yet)
    // history of the second-order scheme: u and F in the lane's own order
    T *const hist = it.hist ? it.hist + lane * 4 : nullptr;
#pragma unroll
    for (int hb = 0; hb < NS; ++hb) {
        V uh = V(T(0)), fh = V(T(0)), un, fn;
        T *const hu = hist + (size_t)hb * 512, *const hf = hu + 256;
        if (hist && !a.first) {
            uh = mm_load(hu);
            fh = mm_load(hf);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const T own = x[hb][i], oth = dpp_mov<ROR8>((T)x[hb][i]);
            const T F = react(own, oth), ud = own - c0;
            T q;
            if (hist) q = fma(a.kc, fma(a.k2, F, -fh[i]), fma(a.k4, ud, -(uh[i] - cp)) * a.kt);
            else q = fma(a.kc, F, ud);
            un[i] = own;
            fn[i] = F;
            if constexpr (RAG) {                              // padding carries no value (and no NaN) on
                if (!real(hb, i)) q = T(0);
            }
            x[hb][i] = q;
        }
        if (hist) {
            *reinterpret_cast<V *>(hu) = un;
            *reinterpret_cast<V *>(hf) = fn;
        }
    }
    L.fwd(x, X);
#pragma unroll
    for (int hb = 0; hb < NS; ++hb) *reinterpret_cast<V *>(row + hb * 16) = X[hb];
}

template <typename T, typename Line>
__device__ __forceinline__ void column_pass(const SplitArgs<T> &a, const SplitItem<T> &it)
{
    using V = Vec4<T>;
    constexpr int N = Line::N, NS = Line::NS;
    const int lane = threadIdx.x, c = lane & 15, sp = c >> 3, g4 = 4 * (lane >> 4);
    Line L;
    L.init(it.cst, lane);
    const auto wb = make_rsrc(it.work, 2u * N * N * sizeof(T));
    const unsigned col = (unsigned)((sp * N + g4) * N + 8 * it.tile + (c & 7)) * (unsigned)sizeof(T);   // its column's slots g4 ..
    const T *dp = (a.first ? it.div : it.div2) + lane * 4;
    V x[NS], X[NS], dv[NS];
    // the column of the rows' means, as in mm_solve: the tiles' constants and the field's
    [[maybe_unused]] float ct[NS], cf = 0.0f;
    [[maybe_unused]] bool differ = false;
    if constexpr (sizeof(T) == 4) {
        if (a.ct && it.tile == 0) {
            bool all = true;
#pragma unroll
            for (int hb = 0; hb < NS; ++hb) {
                ct[hb] = a.ct[(2 * it.k + sp) * 16 + 2 * hb + (lane >> 5)];
                all = all && ct[hb] != 0.0f;
            }
            // (the other half of the species' tiles is 32 lanes on)
            cf = __shfl_xor((int)all, 32, 64) && all ? ct[0] : 0.0f;
#pragma unroll
            for (int hb = 0; hb < NS; ++hb) differ = differ || ct[hb] != cf;
            if ((lane & ~8) == 0) a.c0[2 * it.k + sp] = cf;
        }
    }
#pragma unroll
    for (int hb = 0; hb < NS; ++hb)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[hb][i] = buf_load<T>(wb, col, (hb * 16 + i) * N * (int)sizeof(T));
    auto divisors = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int hb = 0; hb < NS; ++hb) dv[hb] = mm_load(dp + hb * 256);
    };
    if constexpr (sizeof(T) == 4) {
        if (__ballot(differ)) {
#pragma unroll
            for (int hb = 0; hb < NS; ++hb) {
                unsigned rows = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    rows |= ((c & 7) == 0 && slot_valid<Line>(hb, g4 + i, it.s.n) ? 1u : 0u) << i;
                x[hb] = join_offsets(x[hb], (float)it.s.n, ct[hb], cf, rows);
            }
        }
    }
    if constexpr (NS < 8) divisors();                         // ahead of the transform where registers are left
    L.fwd(x, X);
    if constexpr (NS >= 8) divisors();
#pragma unroll
    for (int hb = 0; hb < NS; ++hb) X[hb] *= dv[hb];
    L.inv(X, x);
#pragma unroll
    for (int hb = 0; hb < NS; ++hb)
#pragma unroll
        for (int i = 0; i < 4; ++i) buf_store<T>((T)x[hb][i], wb, col, (hb * 16 + i) * N * (int)sizeof(T));
}

template <int MODEL, typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_tile_rows(SplitArgs<T> a)
{
    const SplitItem<T> it = a.items[blockIdx.x];
    if (it.b < 0) return;
    split_dispatch<T>(it.s.n, [&](auto line) __attribute__((always_inline)) {
        row_pass<MODEL, T, decltype(line)>(a, it);
    });
}

template <typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_tile_columns(SplitArgs<T> a)
{
    const SplitItem<T> it = a.items[blockIdx.x];
    if (it.b < 0) return;
    split_dispatch<T>(it.s.n, [&](auto line) __attribute__((always_inline)) { column_pass<T, decltype(line)>(a, it); });
}

}  // namespace

void split_offsets(int model, const double *p, float (&u0)[2], float (&least)[2])
{
    dispatch_model(model, [&](auto MD) {
        for (int sp = 0; sp < 2; ++sp) {
            StepOffset<decltype(MD)::value> o;
            o.init(p, sp);
            u0[sp] = o.u0;
            least[sp] = o.least;
        }
    });
}

// K steps of the items from the states; from_start: the first of them is the
// second-order scheme's first, an IMEX-Euler step.
template <typename T>
int launch_split(SplitArgs<T> a, int nitems, int model, double dt, int K, bool bdf, bool from_start, hipStream_t st)
{
    auto rows = [&](int flags, bool first) {
        SplitArgs<T> r = a;
        r.flags = flags;
        r.first = first;
        if (bdf && !first) {                                  // as mm_solve's second-order steps
            r.k4 = T(4);
            r.kt = T(1.0 / 3.0);
            r.k2 = T(2);
            r.kc = T(2.0 * dt / 3.0);
        } else {
            r.k4 = r.kt = r.k2 = T(1);
            r.kc = T(dt);
        }
        dispatch_model(model, [&](auto MD) {
            hipLaunchKernelGGL((k_tile_rows<decltype(MD)::value, T>), dim3(nitems), dim3(64), 0, st, r);
        });
    };
    for (int k = 0; k < K; ++k) {
        const bool first = !bdf || (from_start && k == 0);
        if (k == 0) rows(SPLIT_LOAD | SPLIT_NEXT, first);
        SplitArgs<T> q = a;
        q.first = first;
        hipLaunchKernelGGL((k_tile_columns<T>), dim3(nitems), dim3(64), 0, st, q);
        // the state of the step before the last is what the stop rule compares with
        if (k < K - 1) rows(SPLIT_NEXT | (k == K - 2 ? SPLIT_STORE : 0), !bdf);
        else rows(SPLIT_CHECK | SPLIT_STORE, !bdf);
    }
    return check_launch("k_split");
}
template int launch_split<double>(SplitArgs<double>, int, int, double, int, bool, bool, hipStream_t);
template int launch_split<float>(SplitArgs<float>, int, int, double, int, bool, bool, hipStream_t);

}  // namespace cil
