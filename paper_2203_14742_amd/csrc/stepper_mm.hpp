// The matrix-core persistent stepper (templates): one workgroup per solve,
// every grid line transformed on the matrix cores (dct_mfma.hpp).
//
// Work split.  A wavefront owns eight grid lines of both species - the 16
// columns of its MFMA tiles, lanes with l % 16 < 8 species v, the others w, so
// that lane l ^ 8 (a rotation by eight within the row of 16 lanes) holds the
// other species at the same points.  n/8 wavefronts cover the grid.  The field
// lives in LDS in slot order, [species][row slot][column slot], rows padded by
// four values and the species' planes eight values apart: the column pass's
// strided accesses fall on distinct banks; of the row pass's 16-byte ones species
// v of line k + 2 shares banks with species w of line k (32 conflict cycles per
// wavefront and step at 64^2 in FP32 and 128 at 128^2, 1 to 2 % of a step).
// One step is two passes, each in place on the wavefront's own lines and each
// ending with the workgroup barrier:
//   row pass     row inverse (u^s in registers), stop rule and snapshot at
//                evaluation steps, explicit reaction, row forward;
//   column pass  column forward, spectral divide, column inverse.
// The constants of the transforms and (where they fit) the divisors stay in
// registers from the first step to the last.
//
// What bounds it: issue.  FP32 and FP64 matrix and vector instructions of one SIMD
// do not overlap on gfx950 (measured: their times add), so a step costs its
// products (a 64^2 solve in FP32: 64 of 32 cycles per wavefront) plus the folds,
// rotations and reaction.
#pragma once

#include "dct_mfma.hpp"
#include "dct_quad.hpp"
#include "stepper_common.hpp"

namespace cil {

// The reaction of the lane's own species, F = f (sp = 0) or g (sp = 1), from
// its own value and the other species', with per-lane coefficients so that
// both kinds of lane run the same instructions.
template <int MODEL, typename T>
struct OwnReaction {
    T A, B, C;
    bool w;
    __device__ __forceinline__ void init(const double *p, int sp)
    {
        w = sp != 0;
        A = B = C = T(0);
        if constexpr (MODEL == CIL_FHN) {               // A other + (B + C own^2) own
            A = w ? T(-1) : T(p[1]);
            B = w ? T(p[0]) : T(-p[1] * p[2]);
            C = w ? T(-1) : T(0);
        } else if constexpr (MODEL == CIL_GM) {         // B own + v^2 (1/w or 1)
            B = w ? T(-p[1]) : T(-p[0]);
        } else if constexpr (MODEL == CIL_GM_SOURCE) {  // A + B own + v^2 (1/w or 1)
            A = w ? T(0) : T(p[0]);
            B = w ? T(-1) : T(-p[1]);
        } else if constexpr (MODEL == CIL_BRUSSELATOR) {   // A + B v + C v^2 w
            A = w ? T(0) : T(p[0]);
            B = w ? T(p[1]) : T(-(p[1] + 1.0));
            C = w ? T(-1) : T(1);
        }
    }
    __device__ __forceinline__ T operator()(T own, T oth) const
    {
        if constexpr (MODEL == CIL_FHN) {
            return fma(own, fma(C, own * own, B), A * oth);   // (explicit: every kernel rounds it alike)
        } else if constexpr (MODEL == CIL_GM || MODEL == CIL_GM_SOURCE) {
            const T v = w ? oth : own;
            const T r = w ? T(1) : recip(oth);
            return fma(v * v, r, fma(B, own, A));
        } else if constexpr (MODEL == CIL_BRUSSELATOR) {
            const T v = w ? oth : own, z = w ? own : oth;
            return fma(C, v * v * z, fma(B, v, A));
        } else {
            return T(0);
        }
    }
};

// The homogeneous steady state of the lane's species (Sec. 4.1), or 0.  The
// diffusion solve leaves a constant as it is, so FP32 transforms act on
// u - u* instead of u where u is of the size of u*: their rounding is then
// relative to the pattern's amplitude and not to its mean (largest error of 100
// steps near u*: 5e-7 of the field against 4e-6).  Where parts of the field are far
// smaller than u* that would cost their digits, and they act on u.
// A step chooses from the state it starts from and nothing else, so that an
// IMEX-Euler run cut anywhere and carried on from its state rounds as the whole
// run does.  Every tile of eight rows chooses for itself (StepOffset); the field
// between the passes leaves out u* if all tiles do, else 0, and the column of the
// rows' means takes up the difference where a tile chose otherwise (join_offsets).
template <int MODEL>
__host__ __device__ __forceinline__ double steady_value(const double *p, int sp)
{
    double v = 0.0, w = 0.0;
    if constexpr (MODEL == CIL_GM) {
        v = p[1] / p[0];
        w = p[1] / (p[0] * p[0]);
    } else if constexpr (MODEL == CIL_GM_SOURCE) {
        v = (p[0] + 1.0) / p[1];
        w = v * v;
    } else if constexpr (MODEL == CIL_BRUSSELATOR) {
        v = p[0];
        w = p[1] / p[0];
    }
    return sp ? w : v;
}

// Whether a kernel leaves a constant out of its transforms.
template <int MODEL, typename T>
constexpr bool kOffset = sizeof(T) == 4 && MODEL != CIL_FHN && MODEL != CIL_HEAT;

// A step's choice for one tile: u0 = u* if every |u| of it is at least |u*| / 4.
template <int MODEL>
struct StepOffset {
    float u0, least;
    __host__ __device__ __forceinline__ void init(const double *p, int sp)
    {
        const double u = steady_value<MODEL>(p, sp), q = 0.25 * fabs(u);
        const bool ok = fabs(u) <= (double)__FLT_MAX__;                      // (a NaN is none)
        u0 = ok ? (float)u : 0.0f;
        least = ok ? (float)q : __builtin_nanf("");                          // NaN: never
        if ((double)least < q) least = __builtin_bit_cast(float, __builtin_bit_cast(int, least) + 1);     // least float >= q
    }
    // the lanes' species (bit 0: v, bit 1: w) whose values in the tile all reach
    // `least`; abs(hb, i): the lane's values, infinite for padding (any, where the
    // lane's whole row is: `row` false)
    template <int NS, typename F>
    __device__ __forceinline__ unsigned species(bool row, F &&abs) const
    {
        float part[4], m;
#pragma unroll
        for (int i = 0; i < 4; ++i) {                        // four chains side by side
            part[i] = __builtin_inff();
#pragma unroll
            for (int hb = 0; hb < NS; ++hb) part[i] = fminf(part[i], abs(hb, i));
        }
        m = fminf(fminf(part[0], part[1]), fminf(part[2], part[3]));
        const unsigned long long b = __ballot(row && !(m >= least)), v = 0x00FF00FF00FF00FFull;      // lanes of species v
        return ((b & v) ? 0u : 1u) | ((b & ~v) ? 0u : 2u);
    }
};
// Rows' means (column slot 0, unnormalised: n times the mean), x from a tile that
// left out ct to a field that leaves out cf.  Bit i of `rows`: x[i] is the mean of
// a row (not of padding, which a fold adds to the middle row of an odd side).
__device__ __forceinline__ Vec4<float> join_offsets(Vec4<float> x, float n, float ct, float cf, unsigned rows)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = (rows >> i & 1u) && ct != cf ? fmaf(n, ct - cf, x[i]) : x[i];
    return x;
}

// TPW: tiles of eight lines per wavefront (tile = wavefront + WAVES k).  Two
// tiles share one copy of the constants and give the matrix cores independent
// products from one wavefront.
template <typename T, typename Line, int TPW>
struct MmShape {
    static constexpr int N = Line::N, NS = Line::NS;          // N: padded side
    // lines from one tile that is formed to the next: 8, or 16 where every second tile is padding
    static constexpr int PITCH = Line::kShort ? 16 : 8;
    static constexpr int WAVES = N / (PITCH * TPW), THREADS = 64 * WAVES;
    static constexpr int LD = N + 4, SP = N * LD + 8;         // LDS strides, in values
    static constexpr int LDS = 2 * SP;
    // divisors in registers: 4 NS values a lane, where that is at most 16 VGPRs;
    // else read in each step, ahead of the barrier where there is room for them
    // beside the transform's two fields, after the forward where there is not
    static constexpr bool DREG = TPW * NS * sizeof(T) <= 16, DLATE = Line::kRagged && NS * sizeof(T) >= 24;
};

// One solve.  SCHEME 0: IMEX Euler (divisors dtab); 1: the second-order scheme
// (dtab for the first step of the call, dtab2, built with 2 dt / 3, for the
// others; u^{s-2} and F(u^{s-2}) in registers).  The lane's values of u live in
// x: loaded from `state` first when LOAD, stored to `out` (element type TS) at
// the end.  `step` enters as the first step and leaves as the last; returns
// the status of the last evaluation (-1 if none ran).
//
// RF: the refinement form u = U + v (k_fused_q's, stepper_quad.hpp): U in FP64
// in u64, the FP32 correction v in x, R = f(U) + nu Lap U rounded to FP32 in
// LDS behind the field (lane-major, 16 bytes a lane).  Lap U is formed in FP64
// from one species' U at a time, staged in the LDS of the field.
template <typename T, typename Line, int TPW, int MODEL, int SCHEME, bool RF, bool LOAD, typename TS, bool SNAP = false>
__device__ __forceinline__ int mm_solve(T *sm, double *red, int *sbad, const DevSolve &s, int b, T *state, TS *out,
                                        const T *dtab, const T *dtab2, const T *cst, double dt, const PersistArgs &pa,
                                        long long &step, Vec4<T> (&x)[TPW][Line::NS], double *u64 = nullptr)
{
    static_assert(!RF || (std::is_same<T, float>::value && SCHEME == 0 && !Line::kRagged), "");
    using V = Vec4<T>;
    using SH = MmShape<T, Line, TPW>;
    constexpr int NS = Line::NS, LD = SH::LD, SP = SH::SP, WAVES = SH::WAVES, THREADS = SH::THREADS;
    constexpr int PITCH = SH::PITCH, TILE = PITCH / 8 * NS * 256;     // TILE: divisors from wavefront to wavefront
    constexpr bool RAG = Line::kRagged;
    constexpr int ROR8 = 0x128;                               // DPP: rotate by 8 within 16 lanes
    constexpr int STEP = PITCH * WAVES;                       // lines between a wavefront's tiles
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, sp = c >> 3, g4 = 4 * (lane >> 4);
    const int line = PITCH * wave + (c & 7);                  // the lane's row (and column) slot in its first tile
    const int n = RAG ? s.n : Line::N;
    const int NN = n * n;
    Line L;
    L.init(cst, lane);
    OwnReaction<MODEL, T> react;
    react.init(s.p, sp);
    const T tdt = T(dt);
    T *const row = sm + sp * SP + line * LD + g4;             // slots hb * 16 + g4 + i of the lane's row
    T *const col = sm + sp * SP + g4 * LD + line;             // the same of its column, stride LD
    const size_t dsz = (size_t)2 * SH::N * SH::N;
    const T *dp = dtab + s.tab * dsz + (size_t)wave * TILE + lane * 4;
    const T *dp2 = SCHEME ? dtab2 + s.tab * dsz + (size_t)wave * TILE + lane * 4 : dp;
    const auto ub = make_rsrc(state + s.off, 2u * NN * sizeof(T));

    // Element offset of slot (hb, i) of tile k within the solve's state; -1:
    // padding.  `at` is the lane's base, taken anew by each user: the offsets
    // are then formed where they are used instead of being kept in registers
    // across the step loop.
    struct Base {
        int e, g, rn;
        bool ok;
    };
    auto element_base = [&](int k) __attribute__((always_inline)) {
        int ln = line + STEP * k, g = g4;
        asm volatile("" : "+v"(ln), "+v"(g));
        const int rn = slot_pos<Line>(ln >> 4, ln & 15, n);   // the lane's grid row
        return Base{(sp * n + rn) * n, g, rn, slot_valid<Line>(ln >> 4, ln & 15, n)};
    };
    auto elem = [&](const Base &at, int hb, int i) __attribute__((always_inline)) -> int {
        const int e = at.e + slot_pos<Line>(hb, at.g + i, n);
        if constexpr (RAG) return at.ok && slot_valid<Line>(hb, at.g + i, n) ? e : -1;
        else return e;
    };
    // padding carries no value (and no NaN) into the transforms: masks of the lane's real slots
    unsigned real[TPW] = {};
    if constexpr (RAG) {
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            const Base at = element_base(k);
#pragma unroll
            for (int hb = 0; hb < NS; ++hb)
#pragma unroll
                for (int i = 0; i < 4; ++i) real[k] |= (elem(at, hb, i) >= 0 ? 1u : 0u) << (hb * 4 + i);
        }
    }
    auto masked = [&](T v, unsigned bits, int j) __attribute__((always_inline)) -> T {
        const int m = __builtin_amdgcn_sbfe((int)bits, j, 1);
        if constexpr (sizeof(T) == 8)
            return __hiloint2double(__double2hiint(v) & m, __double2loint(v) & m);
        else
            return __int_as_float(__float_as_int(v) & m);
    };
    // the rows of tiles that are not formed stay zero: the constants' zero rows keep them
    if constexpr (Line::kShort) {
#pragma unroll
        for (int hb = 0; hb < NS; ++hb) *reinterpret_cast<V *>(row + 8 * LD + hb * 16) = V(T(0));
    }
    // f(k, hb, i, element) over the lane's slots
    auto each = [&](auto &&f) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            const Base at = element_base(k);
#pragma unroll
            for (int hb = 0; hb < NS; ++hb)
#pragma unroll
                for (int i = 0; i < 4; ++i) f(k, hb, i, elem(at, hb, i));
        }
    };
    // padding reads 0 and is not written (its offset lies past the resource)
    auto ld = [&](auto rsrc, auto type, int e) __attribute__((always_inline)) {
        using E = decltype(type);
        return buf_load<E>(rsrc, e < 0 ? 0xFFFFFF00u : (unsigned)e * (unsigned)sizeof(E), 0);
    };
    auto stv = [&](auto rsrc, auto v, int e) __attribute__((always_inline)) {
        using E = decltype(v);
        buf_store<E>(v, rsrc, e < 0 ? 0xFFFFFF00u : (unsigned)e * (unsigned)sizeof(E), 0);
    };
    if constexpr (LOAD) each([&](int k, int hb, int i, int e) { x[k][hb][i] = ld(ub, T(0), e); });
    // constant the transforms leave out in this step (FP32 without a correction form)
    constexpr bool OFF = kOffset<MODEL, T> && !RF;
    T c0 = T(0);
    [[maybe_unused]] std::conditional_t<OFF, StepOffset<MODEL>, int> offset;
    if constexpr (OFF) offset.init(s.p, sp);
    uint8_t *const chose = reinterpret_cast<uint8_t *>(sbad + WAVES);          // OFF: the tiles' species(), a byte each
    constexpr int DT = WAVES * TILE;                          // divisors between a wavefront's tiles
    V dv[TPW][NS];
    auto load_div = [&](const T *p, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int hb = 0; hb < NS; ++hb) dv[k][hb] = mm_load(p + k * DT + hb * 256);
    };
    if constexpr (SH::DREG) {
#pragma unroll
        for (int k = 0; k < TPW; ++k) load_div(dp, k);
    }
    // refinement form
    V u32[RF ? TPW : 1][RF ? NS : 1];
    V *const rq = RF ? reinterpret_cast<V *>(sm + SH::LDS) + tid : nullptr;
    const auto u64r = make_rsrc(RF ? u64 + s.off : nullptr, RF ? 2u * NN * sizeof(double) : 0);
    auto rebase = [&](bool first) __attribute__((always_inline)) {
        if constexpr (RF) {
            constexpr int DL = Line::N + 1;                   // row stride of the staged FP64 field
            static_assert(Line::N * DL * sizeof(double) <= SH::LDS * sizeof(T), "one FP64 species fits the field");
            double *const sd = reinterpret_cast<double *>(sm);
            double U[TPW][NS][4], lap[TPW][NS][4];
            each([&](int k, int hb, int i, int e) {
                U[k][hb][i] = (double)x[k][hb][i];
                if (!first) U[k][hb][i] += ld(u64r, 0.0, e);
                stv(u64r, U[k][hb][i], e);
                x[k][hb][i] = T(0);
            });
            for (int q = 0; q < 2; ++q) {
                __syncthreads();                              // the LDS's last readers are done
                if (sp == q) {
#pragma unroll
                    for (int k = 0; k < TPW; ++k) {
                        const Base at = element_base(k);
#pragma unroll
                        for (int hb = 0; hb < NS; ++hb)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                sd[at.rn * DL + slot_pos<Line>(hb, at.g + i, n)] = U[k][hb][i];
                    }
                }
                __syncthreads();
                if (sp == q) {
#pragma unroll
                    for (int k = 0; k < TPW; ++k) {
                        const Base at = element_base(k);
                        const int rn = at.rn, ru = rn > 0 ? rn - 1 : 0, rd = rn < n - 1 ? rn + 1 : n - 1;
#pragma unroll
                        for (int hb = 0; hb < NS; ++hb)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int p = slot_pos<Line>(hb, at.g + i, n);
                                const int pl = p > 0 ? p - 1 : 0, pr = p < n - 1 ? p + 1 : n - 1;
                                lap[k][hb][i] = (sd[rn * DL + pl] + sd[rn * DL + pr] + sd[ru * DL + p] +
                                                 sd[rd * DL + p] - 4.0 * U[k][hb][i]) * s.inv_h2;
                            }
                    }
                }
            }
            const double pd[4] = {s.p[0], s.p[1], s.p[2], s.p[3]}, nu = sp ? s.nu[1] : s.nu[0];
#pragma unroll
            for (int k = 0; k < TPW; ++k)
#pragma unroll
                for (int hb = 0; hb < NS; ++hb) {
                    V r;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const double Us = U[k][hb][i], Uo = dpp_mov<ROR8>(U[k][hb][i]);
                        double f, gg;
                        kinetics<MODEL>(pd, sp ? Uo : Us, sp ? Us : Uo, f, gg);
                        r[i] = (T)((sp ? gg : f) + nu * lap[k][hb][i]);
                        u32[k][hb][i] = (T)Us;
                    }
                    rq[(k * NS + hb) * THREADS] = r;          // read back by this lane alone
                }
            __syncthreads();                                  // the FP64 field's last readers are done
        }
    };
    // second order: r = kt (k4 u^{s-1} - u^{s-2}) + kc (k2 F(u^{s-1}) - F(u^{s-2})) with (k4, kt, k2, kc) = (4, 1/3,
    // 2, 2 dt / 3); the first step is the IMEX-Euler one, (1, 1, 1, dt) and an empty history
    V uh[SCHEME ? TPW : 1][SCHEME ? NS : 1] = {}, fh[SCHEME ? TPW : 1][SCHEME ? NS : 1] = {};
    T k4 = T(1), kt = T(1), k2 = T(1), kc = tdt;
    const T *dsel = dp;                                       // the divisors of the step
    long long last_rebase = step;
    if constexpr (RF) rebase(true);
    // the stop rule's snapshot of the step before an evaluation: in registers (SNAP), or in the state
    static_assert(!SNAP || (TPW == 1 && SCHEME == 0 && !RAG && !RF), "");
    V snap[SNAP ? NS : 1];
    int fin = -1;
    while (step < pa.max_steps) {
        // up to the next evaluation step, whose predecessor is kept as the stop rule's snapshot
        const long long stop = (step / pa.check + 1) * pa.check;
        const long long upto = stop < pa.max_steps ? stop : pa.max_steps;
        int left = (int)(upto - step);                        // at most check_every
        step = upto;
        while (true) {
            if (left == 1) {
                if constexpr (SNAP) {
#pragma unroll
                    for (int hb = 0; hb < NS; ++hb) snap[hb] = x[0][hb];
                } else {
                    each([&](int k, int hb, int i, int e) { stv(ub, (T)x[k][hb][i], e); });
                }
            }
#pragma unroll
            for (int k = 0; k < TPW; ++k) {
                // explicit reaction
                V X[NS];
                if constexpr (OFF) {
                    const bool isrow = !RAG || (real[k] & 1u);       // (slot 0 is a position of every row)
                    const unsigned has = offset.template species<NS>(isrow, [&](int hb, int i) __attribute__((always_inline)) {
                        return slot_full<Line>(hb) || (real[k] >> (hb * 4 + i) & 1u) ? fabsf(x[k][hb][i]) : __builtin_inff();
                    });
                    chose[wave + WAVES * k] = (uint8_t)has;       // (every lane: no branch)
                    c0 = (has >> sp) & 1u ? offset.u0 : 0.0f;
                }
#pragma unroll
                for (int hb = 0; hb < NS; ++hb) {
                    V r;
                    if constexpr (RF) r = rq[(k * NS + hb) * THREADS];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const T own = x[k][hb][i], oth = dpp_mov<ROR8>((T)x[k][hb][i]);
                        T q;
                        if constexpr (RF) {                   // v + dt (R + f(U + v) - f(U))
                            const T ua = u32[k][hb][i], uo = dpp_mov<ROR8>((T)u32[k][hb][i]);
                            T f, gg;
                            const T p[4] = {T(s.p[0]), T(s.p[1]), T(s.p[2]), T(s.p[3])};
                            kinetics_delta<MODEL>(p, sp ? uo : ua, sp ? ua : uo, sp ? oth : own, sp ? own : oth, f, gg);
                            q = own + tdt * (r[i] + (sp ? gg : f));
                        } else if constexpr (SCHEME == 1) {
                            const T F = react(own, oth), ud = own - c0;
                            const T up = uh[k][hb][i] - (dsel == dp2 ? c0 : T(0));        // (first step: none)
                            q = fma(kc, fma(k2, F, -fh[k][hb][i]), fma(k4, ud, -up) * kt);
                            uh[k][hb][i] = own;
                            fh[k][hb][i] = F;
                        } else {
                            q = fma(tdt, react(own, oth), own - c0);
                        }
                        if constexpr (RAG) q = masked(q, real[k], hb * 4 + i);
                        x[k][hb][i] = q;
                    }
                }
                L.fwd(x[k], X);
#pragma unroll
                for (int hb = 0; hb < NS; ++hb) *reinterpret_cast<V *>(row + STEP * LD * k + hb * 16) = X[hb];
            }
            if constexpr (!SH::DREG && !SH::DLATE) load_div(dsel, 0);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < TPW; ++k) {
                V X[NS];
#pragma unroll
                for (int hb = 0; hb < NS; ++hb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[k][hb][i] = col[STEP * k + (hb * 16 + i) * LD];
                if constexpr (!SH::DREG && !SH::DLATE) {
                    if (k > 0) load_div(dsel, k);
                }
                if constexpr (OFF) {
                    if (k == 0) {                             // (behind the column's reads: its latency is theirs)
                        constexpr int TILES = WAVES * TPW;
                        const unsigned ones = TILES == 2 ? 0x0101u : 0x01010101u;
                        unsigned any = 0, all = ~0u;
                        if constexpr (TILES == 2) {
                            any = all = *reinterpret_cast<const uint16_t *>(chose);
                        } else {
#pragma unroll
                            for (int w = 0; w < TILES / 4; ++w) {
                                const unsigned f = (unsigned)sbad[WAVES + w];
                                any |= f;
                                all &= f;
                            }
                        }
                        c0 = (all & (ones << sp)) == ones << sp ? offset.u0 : 0.0f;
                        if (__builtin_amdgcn_readfirstlane(wave) == 0) {
                            any = __builtin_amdgcn_readfirstlane(any);
                            all = __builtin_amdgcn_readfirstlane(all);
                            // some tile left out another constant than the field
                            if (((any & ones) && (all & ones) != ones) || ((any & 2 * ones) && (all & 2 * ones) != 2 * ones)) {
#pragma unroll
                                for (int hb = 0; hb < NS; ++hb) {         // the lane's rows are of tile 2 hb + g / 2
                                    const int t = (2 * hb + (lane >> 5)) / (PITCH / 8);
                                    const float ct = (chose[t] >> sp) & 1u ? offset.u0 : 0.0f;
                                    const unsigned rows = (c & 7) != 0 ? 0u : RAG ? real[0] >> (4 * hb) : 15u;     // (their own slots)
                                    x[k][hb] = join_offsets(x[k][hb], (float)n, ct, c0, rows);
                                }
                            }
                        }
                    }
                }
                L.fwd(x[k], X);
                if constexpr (SH::DLATE) load_div(dsel, k);
#pragma unroll
                for (int hb = 0; hb < NS; ++hb) X[hb] *= dv[k][hb];
                L.inv(X, x[k]);
#pragma unroll
                for (int hb = 0; hb < NS; ++hb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) col[STEP * k + (hb * 16 + i) * LD] = x[k][hb][i];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < TPW; ++k) {
                V X[NS];
#pragma unroll
                for (int hb = 0; hb < NS; ++hb) X[hb] = *reinterpret_cast<const V *>(row + STEP * LD * k + hb * 16);
                L.inv(X, x[k]);
                if constexpr (kOffset<MODEL, T> && !RF) {
#pragma unroll
                    for (int hb = 0; hb < NS; ++hb) x[k][hb] += V(c0);
                }
            }
            if constexpr (SCHEME == 1) {
                if (dsel != dp2) {
                    dsel = dp2;
                    k4 = T(4);
                    kt = T(1.0 / 3.0);                        // a multiply, not a divide
                    k2 = T(2);
                    kc = T(2.0 * dt / 3.0);
                    if constexpr (SH::DREG) {
#pragma unroll
                        for (int k = 0; k < TPW; ++k) load_div(dp2, k);
                    }
                }
            }
            if (--left == 0) break;
        }
        // stop rule on u^step against the snapshot of u^(step-1)
        double d = 0.0, a = 0.0;
        int bad = 0;
        each([&](int k, int hb, int i, int e) {
            const double v = (double)x[k][hb][i];
            double before;
            if constexpr (SNAP) before = (double)snap[hb][i];
            else before = (double)ld(ub, T(0), e);
            const double dd = fabs(v - before);
            if (!RAG || e >= 0) {
                bad |= !isfinite(v);
                d = fmax(d, isnan(dd) ? 0.0 : dd);
                if constexpr (!RF) a = fmax(a, isnan(v) ? 0.0 : fabs(v));
            }
        });
        d = wave_max(d);
        a = wave_max(a);
        bad = wave_or(bad);
        if (lane == 0) {
            red[wave] = d;
            red[WAVES + wave] = a;
            sbad[wave] = bad;
        }
        __syncthreads();
        double dm = 0.0, am = 0.0;
        int anybad = 0;
        for (int w = 0; w < WAVES; ++w) {
            dm = fmax(dm, red[w]);
            am = fmax(am, red[WAVES + w]);
            anybad |= sbad[w];
        }
        const double r = dm / dt;
        int st = -1;
        if (anybad) st = CIL_SOLVE_NONFINITE;
        else if (pa.tol > 0.0 && r < pa.tol) st = CIL_SOLVE_OK;
        else if (pa.tol > 0.0 && pa.floor_coef > 0.0 && r < pa.floor_coef * am) st = CIL_SOLVE_FP32_FLOOR;
        else if (step == pa.max_steps) st = pa.tol > 0.0 ? CIL_SOLVE_MAXSTEPS : CIL_SOLVE_OK;
        if (tid == 0) {
            pa.resid[b] = anybad ? (double)NAN : r;
            if (st >= 0) pa.status[b] = st;
        }
        fin = st;
        if (st >= 0) break;
        if (pa.prio > 1.0 && pa.tol > 0.0) set_issue_priority(r / pa.tol, pa.prio);
        if constexpr (RF) {
            if (step - last_rebase >= kRebase) {          // uniform over the workgroup
                rebase(false);
                last_rebase = step;
            }
        }
    }
    const auto ob = make_rsrc(out + s.off, 2u * NN * sizeof(TS));
    each([&](int k, int hb, int i, int e) {
        if constexpr (RF) x[k][hb][i] = T(ld(u64r, 0.0, e) + (double)x[k][hb][i]);     // u = U + v
        stv(ob, TS(x[k][hb][i]), e);
    });
    if (tid == 0) pa.steps[b] = step;
    return fin;
}

// One kernel per model (the host picks it).  WPE: wavefronts per SIMD that the
// register allocation aims at.
template <int MODEL, typename T, typename Line, int SCHEME, int TPW, int WPE, bool SNAP>
__global__ __launch_bounds__((MmShape<T, Line, TPW>::THREADS)) __attribute__((amdgpu_waves_per_eu(WPE))) void k_mm(
    const DevSolve *S, const int *list, T *state, const T *dtab, const T *dtab2, const T *cst, double dt,
    PersistArgs pa)
{
    using SH = MmShape<T, Line, TPW>;
    __shared__ __align__(16) T sm[SH::LDS];
    __shared__ double red[2 * SH::WAVES];
    __shared__ int sbad[SH::WAVES + 4];
    const int b = list[blockIdx.x];
    const DevSolve s = S[b];
    long long step = pa.steps[b];
    Vec4<T> x[TPW][Line::NS];
    mm_solve<T, Line, TPW, MODEL, SCHEME, false, true, T, SNAP>(sm, red, sbad, s, b, state, state, dtab, dtab2, cst, dt, pa, step,
                                                     x);
}

// FP32 steps, then from the FP32 floor to the tolerance the refinement form
// (RF) or FP64 steps, in one launch or two: modes and arguments as
// k_fused_q_mixed (stepper_quad.hpp), whose two phases these are on the matrix
// cores.
template <int MODEL, typename LineF, typename LineD, int TPW, int WPE, bool RF>
__global__ __launch_bounds__((MmShape<float, LineF, TPW>::THREADS)) __attribute__((amdgpu_waves_per_eu(WPE)))
void k_mm_mixed(const DevSolve *S, const int *list, float *state, double *state64, const float *tab32,
                const double *tab64, double dt, PersistArgs pa32, PersistArgs pa64, long long *switch_step, int mode)
{
    using SF = MmShape<float, LineF, TPW>;
    using SD = MmShape<double, LineD, TPW>;
    constexpr int N = LineF::N, NS = LineF::NS;
    // the refinement form keeps R behind the field
    __shared__ __align__(16) double sm[RF ? SF::LDS / 2 + N * N : SD::LDS];
    __shared__ double red[2 * SF::WAVES];
    __shared__ int sbad[SF::WAVES + 4];
    const int b = list[blockIdx.x];
    const DevSolve s = S[b];
    long long step = pa32.steps[b];
    if (mode == 2) pa32.max_steps = step;
    Vec4<float> x[TPW][NS];
    const int fin = mm_solve<float, LineF, TPW, MODEL, 0, false, true, float>(
        reinterpret_cast<float *>(sm), red, sbad, s, b, state, state, tab32, nullptr, nullptr, dt, pa32, step, x);
    const long long sw = step;
    const bool go = mode == 2 || (mode == 0 && fin == CIL_SOLVE_FP32_FLOOR);       // uniform over the workgroup
    if constexpr (RF) {
        if (go)
            mm_solve<float, LineF, TPW, MODEL, 0, true, false, float>(reinterpret_cast<float *>(sm), red, sbad, s, b,
                                                                      state, state, tab32, nullptr, nullptr, dt, pa64,
                                                                      step, x, state64);
    } else if (go) {
        Vec4<double> v[TPW][NS];
#pragma unroll
        for (int k = 0; k < TPW; ++k)
#pragma unroll
            for (int hb = 0; hb < NS; ++hb)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[k][hb][i] = (double)x[k][hb][i];
        __syncthreads();                                      // the LDS is reused at double width
        mm_solve<double, LineD, TPW, MODEL, 0, false, false, float>(sm, red, sbad, s, b, state64, state, tab64,
                                                                    nullptr, nullptr, dt, pa64, step, v);
    }
    if (threadIdx.x == 0 && mode != 2) switch_step[b] = sw;
}

// Whether a kernel has a form that keeps the stop rule's snapshot in registers, for
// runs evaluated every few steps (at most kSnapCheck apart): 300 FP64 solves of 64^2
// evaluated at every step 17.5 us a step so, 27.9 through the state; 3000 FP32 ones
// of 32^2 14.3 and 20.5, at every fifth 10.6 and 10.9.  Its registers cost 3 % of
// a step where evaluations are rare.
template <typename T, typename Line, int SCHEME>
constexpr bool kHasSnap = SCHEME == 0 && Line::N == (sizeof(T) == 8 ? 64 : 32) && !Line::kRagged;
constexpr int kSnapCheck = 4;

template <typename T, typename Line, int SCHEME, int TPW, int WPE>
void launch_mm_line(int nl, const DevSolve *S, const int *list, T *state, const T *dtab, const T *dtab2, const T *cst,
                    int model, double dt, const PersistArgs &pa, hipStream_t st)
{
    constexpr int threads = MmShape<T, Line, TPW>::THREADS;
    dispatch_model(model, [&](auto MD) {
        if constexpr (kHasSnap<T, Line, SCHEME>) {
            if (pa.check <= kSnapCheck) {
                hipLaunchKernelGGL((k_mm<decltype(MD)::value, T, Line, SCHEME, TPW, WPE, true>), dim3(nl), dim3(threads), 0,
                                   st, S, list, state, dtab, dtab2, cst, dt, pa);
                return;
            }
        }
        hipLaunchKernelGGL((k_mm<decltype(MD)::value, T, Line, SCHEME, TPW, WPE, false>), dim3(nl), dim3(threads), 0, st, S,
                           list, state, dtab, dtab2, cst, dt, pa);
    });
}

}  // namespace cil
