// Line transforms (DCT-II and its inverse) on the matrix cores.
//
// A wavefront transforms 16 grid lines at once: MFMA 16x16x4 products
// D[16 x 16] += A[16 x 4] B[4 x 16] with a constant 16 x 16 cosine block as A
// and the lines as the columns of B.  Lane l holds column c = l % 16 (its
// line) and, of every block of 16 positions, the four with labels 4 g + i,
// g = l / 16, i = 0..3.  The accumulator of one product has the layout of the
// B operand of the next (only the order of the labels within a block is the
// matrix core's own, and the constant blocks are laid out to match), so a
// whole transform - folds, products, rotations - never leaves the registers.
//
// A line of N values is folded down to 16-point blocks, which the matrix
// cores take as dense products:
//   DCT-II_N   even outputs: DCT-II_{N/2} of x_j + x_{N-1-j},
//              odd outputs: DCT-IV_{N/2} of x_j - x_{N-1-j};
//   DCT-IV_M   with theta_j = pi (2j+1) / 4M and j < M/2: the rotated pairs
//              A_j = a cos + b sin, B_j = b cos - a sin (a = d_j, b =
//              d_{M-1-j}), U = DCT-II_{M/2}(A), V = DST-II_{M/2}(B), then
//              y_{2p} = U_p + V_p, y_{2p-1} = U_p - V_p;
//   DST-II_M   odd p: DST-IV_{M/2} of B_j + B_{M-1-j}, even p: DST-II_{M/2} of
//              B_j - B_{M-1-j}.
// (Chen, Smith and Fralick 1977; Wang 1984.)  For N = 32, 64, 128 that is 2,
// 4, 8 products of 256 multiply-adds per line against N^2 / 256 = 4, 16, 64
// of the dense transform; partners of every fold share a lane, so the folds
// are register adds.  Any other N <= 128 takes the first fold only
// (LineDense), padded to a multiple of 32 with zero rows and columns in the
// constants.  Cosines are unnormalised; the weights 1/n, 2/n of the inverse sit
// in the spectral divisor (so the constant mode's gain over a step is exactly one
// where n is a power of two, elsewhere the rounded 1/n^2 times n^2, the same
// within half a unit in the last place at every step).
//
// Positions and modes are kept in slot order: slot (hb, label) of a line is
// grid position pos(hb, label), and of its spectrum mode(hb, label).
#pragma once

#include "cil_internal.hpp"

namespace cil {

template <typename T>
using Vec4 = T __attribute__((ext_vector_type(4)));

__device__ __forceinline__ Vec4<float> mma4(float a, float b, Vec4<float> c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ Vec4<double> mma4(double a, double b, Vec4<double> c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Label of row r of an MFMA result: lane group g holds rows 4g + i in FP32 and
// g + 4i in FP64, and either way its register i is label 4g + i.
template <typename T>
__host__ __device__ constexpr int mma_row_label(int r)
{
    return sizeof(T) == 8 ? 4 * (r & 3) + (r >> 2) : r;
}

// a b + c on four values.  Written out wherever a product meets a sum, so that
// every kernel that holds a transform rounds it alike.
template <typename T>
__device__ __forceinline__ Vec4<T> fma4(const Vec4<T> &a, const Vec4<T> &b, const Vec4<T> &c)
{
    return __builtin_elementwise_fma(a, b, c);
}

// Two independent 16 x 16 block products, interleaved: a chain of dependent
// FP32 products issues every 56 cycles, two in turn every 36 (measured).
template <typename T>
__device__ __forceinline__ void block2(const Vec4<T> &A0, const Vec4<T> &x0, Vec4<T> &c0, const Vec4<T> &A1,
                                       const Vec4<T> &x1, Vec4<T> &c1)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c0 = mma4(A0[i], x0[i], c0);
        c1 = mma4(A1[i], x1[i], c1);
    }
}

// ------------------------------------------------------------ constants
// 16-point blocks in operand order, mat[k][lane][i] = M_k[row][4 g + i] with
// row = mma_row_label(lane % 16), and the rotations' cosines and sines by
// label.  Index 0 of the DST-II outputs stands for its last one, p = 16.
enum { MM_C2 = 0, MM_C2T, MM_C4, MM_S2, MM_S2T, MM_S4, MM_MATS };

template <typename T>
struct MmConst {
    T mat[MM_MATS][64][4];
    T c32[16], s32[16];           // theta = pi (2j+1) / 128, j = label
    T c64[2][16], s64[2][16];     // theta = pi (2j+1) / 256, j = label and 31 - label
};

// cos(pi t / 256), t = 0..128, correctly rounded: an error of these constants
// is the same at every step, so it adds up over a run.
constexpr double kCos256[129] = {
    1.0, 0x1.fff62169b92dbp-1, 0x1.ffd886084cd0dp-1, 0x1.ffa72effef75dp-1,
    0x1.ff621e3796d7ep-1, 0x1.ff095658e71adp-1, 0x1.fe9cdad01883ap-1, 0x1.fe1cafcbd5b09p-1,
    0x1.fd88da3d12526p-1, 0x1.fce15fd6da67bp-1, 0x1.fc26470e19fd3p-1, 0x1.fb5797195d741p-1,
    0x1.fa7557f08a517p-1, 0x1.f97f924c9099bp-1, 0x1.f8764fa714ba9p-1, 0x1.f7599a3a12077p-1,
    0x1.f6297cff75cb0p-1, 0x1.f4e603b0b2f2dp-1, 0x1.f38f3ac64e589p-1, 0x1.f2252f7763adap-1,
    0x1.f0a7efb9230d7p-1, 0x1.ef178a3e473c2p-1, 0x1.ed740e7684963p-1, 0x1.ebbd8c8df0b74p-1,
    0x1.e9f4156c62ddap-1, 0x1.e817bab4cd10dp-1, 0x1.e6288ec48e112p-1, 0x1.e426a4b2bc17ep-1,
    0x1.e212104f686e5p-1, 0x1.dfeae622dbe2bp-1, 0x1.ddb13b6ccc23cp-1, 0x1.db6526238a09bp-1,
    0x1.d906bcf328d46p-1, 0x1.d696173c9e68bp-1, 0x1.d4134d14dc93ap-1, 0x1.d17e7743e35dcp-1,
    0x1.ced7af43cc773p-1, 0x1.cc1f0f3fcfc5cp-1, 0x1.c954b213411f5p-1, 0x1.c678b3488739bp-1,
    0x1.c38b2f180bdb1p-1, 0x1.c08c426725549p-1, 0x1.bd7c0ac6f952ap-1, 0x1.ba5aa673590d2p-1,
    0x1.b728345196e3ep-1, 0x1.b3e4d3ef55712p-1, 0x1.b090a58150200p-1, 0x1.ad2bc9e21d511p-1,
    0x1.a9b66290ea1a3p-1, 0x1.a63091b02fae2p-1, 0x1.a29a7a0462782p-1, 0x1.9ef43ef29af94p-1,
    0x1.9b3e047f38741p-1, 0x1.9777ef4c7d742p-1, 0x1.93a22499263fbp-1, 0x1.8fbcca3ef940dp-1,
    0x1.8bc806b151741p-1, 0x1.87c400fba2ebfp-1, 0x1.83b0e0bff976ep-1, 0x1.7f8ece3571771p-1,
    0x1.7b5df226aafafp-1, 0x1.771e75f037261p-1, 0x1.72d0837efff96p-1, 0x1.6e74454eaa8afp-1,
    0x1.6a09e667f3bcdp-1, 0x1.6591925f0783dp-1, 0x1.610b7551d2cdfp-1, 0x1.5c77bbe65018cp-1,
    0x1.57d69348ceca0p-1, 0x1.5328292a35596p-1, 0x1.4e6cabbe3e5e9p-1, 0x1.49a449b9b0939p-1,
    0x1.44cf325091dd6p-1, 0x1.3fed9534556d4p-1, 0x1.3affa292050b9p-1, 0x1.36058b10659f3p-1,
    0x1.30ff7fce17035p-1, 0x1.2bedb25faf3eap-1, 0x1.26d054cdd12dfp-1, 0x1.21a799933eb59p-1,
    0x1.1c73b39ae68c8p-1, 0x1.1734d63dedb49p-1, 0x1.11eb3541b4b23p-1, 0x1.0c9704d5d898fp-1,
    0x1.073879922ffeep-1, 0x1.01cfc874c3eb7p-1, 0x1.f8ba4dbf89abap-2, 0x1.edc1952ef78d6p-2,
    0x1.e2b5d3806f63bp-2, 0x1.d79775b86e389p-2, 0x1.cc66e9931c45ep-2, 0x1.c1249d8011ee7p-2,
    0x1.b5d1009e15cc0p-2, 0x1.aa6c82b6d3fcap-2, 0x1.9ef7943a8ed8ap-2, 0x1.9372a63bc93d7p-2,
    0x1.87de2a6aea963p-2, 0x1.7c3a9311dcce7p-2, 0x1.7088530fa459fp-2, 0x1.64c7ddd3f27c6p-2,
    0x1.58f9a75ab1fddp-2, 0x1.4d1e24278e76ap-2, 0x1.4135c94176601p-2, 0x1.35410c2e18152p-2,
    0x1.294062ed59f06p-2, 0x1.1d3443f4cdb3ep-2, 0x1.111d262b1f677p-2, 0x1.04fb80e37fdaep-2,
    0x1.f19f97b215f1bp-3, 0x1.d934fe5454311p-3, 0x1.c0b826a7e4f63p-3, 0x1.a82a025b00451p-3,
    0x1.8f8b83c69a60bp-3, 0x1.76dd9de50bf31p-3, 0x1.5e214448b3fc6p-3, 0x1.45576b1293e5ap-3,
    0x1.2c8106e8e613ap-3, 0x1.139f0cedaf577p-3, 0x1.f564e56a9730ep-4, 0x1.c3785c79ec2d5p-4,
    0x1.917a6bc29b42cp-4, 0x1.5f6d00a9aa419p-4, 0x1.2d52092ce19f6p-4, 0x1.f656e79f820e0p-5,
    0x1.91f65f10dd814p-5, 0x1.2d865759455cdp-5, 0x1.92155f7a3667ep-6, 0x1.921d1fcdec784p-7,
    0.0,
};
constexpr double mm_cos256(int t)
{
    t &= 511;                                             // period 2 pi
    if (t > 256) t = 512 - t;
    return t > 128 ? -kCos256[256 - t] : kCos256[t];
}
constexpr double mm_sin256(int t) { return mm_cos256(t - 128); }

template <typename T>
constexpr MmConst<T> make_mm_const()
{
    MmConst<T> r{};
    auto cosp = [](int t) { return mm_cos256(4 * t); };   // of pi t / 64
    auto sinp = [](int t) { return mm_sin256(4 * t); };
    for (int l = 0; l < 64; ++l)
        for (int i = 0; i < 4; ++i) {
            const int row = mma_row_label<T>(l & 15), col = 4 * (l >> 4) + i;
            const int rs = row ? row : 16, ccs = col ? col : 16;
            r.mat[MM_C2][l][i] = T(cosp(2 * row * (2 * col + 1)));
            r.mat[MM_C2T][l][i] = T(cosp(2 * col * (2 * row + 1)));
            r.mat[MM_C4][l][i] = T(cosp((2 * row + 1) * (2 * col + 1)));
            r.mat[MM_S2][l][i] = T(sinp(2 * rs * (2 * col + 1)));
            r.mat[MM_S2T][l][i] = T(sinp(2 * ccs * (2 * row + 1)));
            r.mat[MM_S4][l][i] = T(sinp((2 * row + 1) * (2 * col + 1)));
        }
    for (int j = 0; j < 16; ++j) {
        r.c32[j] = T(mm_cos256(4 * j + 2));
        r.s32[j] = T(mm_sin256(4 * j + 2));
        r.c64[0][j] = T(mm_cos256(2 * j + 1));
        r.s64[0][j] = T(mm_sin256(2 * j + 1));
        r.c64[1][j] = T(mm_cos256(63 - 2 * j));
        r.s64[1][j] = T(mm_sin256(63 - 2 * j));
    }
    return r;
}

template <typename T>
static __device__ const MmConst<T> kMmConst = make_mm_const<T>();

template <typename T>
__device__ __forceinline__ Vec4<T> mm_load(const T *p)
{
    return *reinterpret_cast<const Vec4<T> *>(p);
}

// ---------------------------------------------------------------- N = 32
template <typename T>
struct Line32 {
    using V = Vec4<T>;
    static constexpr int N = 32, NS = 2;                  // NS: blocks of 16 slots
    static constexpr bool kRagged = false, kShort = false;
    V C2, C2T, C4;
    __device__ __forceinline__ void init(const T *, int lane)
    {
        C2 = mm_load(kMmConst<T>.mat[MM_C2][lane]);
        C2T = mm_load(kMmConst<T>.mat[MM_C2T][lane]);
        C4 = mm_load(kMmConst<T>.mat[MM_C4][lane]);
    }
    __device__ __forceinline__ void fwd(const V (&x)[NS], V (&X)[NS]) const
    {
        const V s = x[0] + x[1], d = x[0] - x[1];
        X[0] = V(T(0));
        X[1] = V(T(0));
        block2<T>(C2, s, X[0], C4, d, X[1]);
    }
    __device__ __forceinline__ void inv(const V (&X)[NS], V (&x)[NS]) const
    {
        V e = V(T(0)), o = V(T(0));
        block2<T>(C2T, X[0], e, C4, X[1], o);
        x[0] = e + o;
        x[1] = e - o;
    }
    // grid position of slot (hb, label): off + label, or off - label
    __host__ __device__ static constexpr bool desc(int hb) { return hb == 1; }
    __host__ __device__ static constexpr int off(int hb) { return hb == 1 ? 31 : 0; }
    __host__ __device__ static constexpr int mode(int hb, int lab) { return 2 * lab + hb; }
};

// ---------------------------------------------------------------- N = 64
// Slots hb = 0..3: positions lab, 31 - lab, 63 - lab, 32 + lab.
template <typename T>
struct Line64 {
    using V = Vec4<T>;
    static constexpr int N = 64, NS = 4;
    static constexpr bool kRagged = false, kShort = false;
    V C2, C2T, C4, S2, S2T, rc, rs;
    T keep;                                               // 0 for label 0 (register 0 of group 0), else 1
    __device__ __forceinline__ void init(const T *, int lane)
    {
        C2 = mm_load(kMmConst<T>.mat[MM_C2][lane]);
        C2T = mm_load(kMmConst<T>.mat[MM_C2T][lane]);
        C4 = mm_load(kMmConst<T>.mat[MM_C4][lane]);
        S2 = mm_load(kMmConst<T>.mat[MM_S2][lane]);
        S2T = mm_load(kMmConst<T>.mat[MM_S2T][lane]);
        rc = mm_load(&kMmConst<T>.c32[4 * (lane >> 4)]);
        rs = mm_load(&kMmConst<T>.s32[4 * (lane >> 4)]);
        keep = lane < 16 ? T(0) : T(1);
    }
    // y_{2p} = U_p + V_p, y_{2p-1} = U_p - V_p; at label 0 y_0 = U_0 and the last output is -V_16
    __device__ __forceinline__ void join(const V &U, const V &W, V &a, V &b) const
    {
        a = U + W;
        b = U - W;
        a[0] = fma(keep, W[0], U[0]);
        b[0] = fma(keep, U[0], -W[0]);
    }
    __device__ __forceinline__ void fwd_regs(const V &x0, const V &x1, const V &x2, const V &x3, V &X0, V &X1, V &X2,
                                             V &X3) const
    {
        const V s0 = x0 + x2, d0 = x0 - x2, s1 = x1 + x3, d1 = x1 - x3;
        const V A = fma4<T>(d0, rc, d1 * rs), B = fma4<T>(d1, rc, -(d0 * rs));
        V U = V(T(0)), W = V(T(0));
        block2<T>(C2, A, U, S2, B, W);
        X0 = V(T(0));
        X1 = V(T(0));
        block2<T>(C2, s0 + s1, X0, C4, s0 - s1, X1);
        join(U, W, X2, X3);
    }
    __device__ __forceinline__ void inv_regs(const V &X0, const V &X1, const V &X2, const V &X3, V &x0, V &x1, V &x2,
                                             V &x3) const
    {
        V U, W;
        join(X2, X3, U, W);
        V A = V(T(0)), B = V(T(0)), e = V(T(0)), o = V(T(0));
        block2<T>(C2T, U, A, S2T, W, B);
        block2<T>(C2T, X0, e, C4, X1, o);
        const V s0 = e + o, s1 = e - o;
        const V d0 = fma4<T>(A, rc, -(B * rs)), d1 = fma4<T>(B, rc, A * rs);
        x0 = s0 + d0;
        x2 = s0 - d0;
        x1 = s1 + d1;
        x3 = s1 - d1;
    }
    __device__ __forceinline__ void fwd(const V (&x)[NS], V (&X)[NS]) const
    {
        fwd_regs(x[0], x[1], x[2], x[3], X[0], X[1], X[2], X[3]);
    }
    __device__ __forceinline__ void inv(const V (&X)[NS], V (&x)[NS]) const
    {
        inv_regs(X[0], X[1], X[2], X[3], x[0], x[1], x[2], x[3]);
    }
    __host__ __device__ static constexpr bool desc(int hb) { return hb == 1 || hb == 2; }
    __host__ __device__ static constexpr int off(int hb) { return hb == 0 ? 0 : hb == 1 ? 31 : hb == 2 ? 63 : 32; }
    __host__ __device__ static constexpr int mode(int hb, int lab)
    {
        return hb == 0 ? 4 * lab : hb == 1 ? 4 * lab + 2 : hb == 2 ? 4 * lab + 1 : lab == 0 ? 63 : 4 * lab - 1;
    }
};

// --------------------------------------------------------------- N = 128
// Slots hb = 0..3 as N = 64 on the first half, hb + 4 their mirrors 127 - j.
template <typename T>
struct Line128 {
    using V = Vec4<T>;
    static constexpr int N = 128, NS = 8;
    static constexpr bool kRagged = false, kShort = false;
    Line64<T> h;
    V S4, rc0, rs0, rc1, rs1;
    __device__ __forceinline__ void init(const T *, int lane)
    {
        h.init(nullptr, lane);
        const int g4 = 4 * (lane >> 4);
        S4 = mm_load(kMmConst<T>.mat[MM_S4][lane]);
        rc0 = mm_load(&kMmConst<T>.c64[0][g4]);
        rs0 = mm_load(&kMmConst<T>.s64[0][g4]);
        rc1 = mm_load(&kMmConst<T>.c64[1][g4]);
        rs1 = mm_load(&kMmConst<T>.s64[1][g4]);
    }
    __device__ __forceinline__ void fwd(const V (&x)[NS], V (&X)[NS]) const
    {
        {
            const V d0 = x[0] - x[4], d2 = x[2] - x[6], d1 = x[1] - x[5], d3 = x[3] - x[7];
            const V A0 = fma4<T>(d0, rc0, d2 * rs0), B0 = fma4<T>(d2, rc0, -(d0 * rs0));
            const V A1 = fma4<T>(d1, rc1, d3 * rs1), B1 = fma4<T>(d3, rc1, -(d1 * rs1));
            V Ue = V(T(0)), Uo = V(T(0)), We = V(T(0)), Wo = V(T(0));
            block2<T>(h.C2, A0 + A1, Ue, h.S2, B0 - B1, We);
            block2<T>(h.C4, A0 - A1, Uo, S4, B0 + B1, Wo);
            const V s0 = x[0] + x[4], s1 = x[1] + x[5], s2 = x[2] + x[6], s3 = x[3] + x[7];
            h.join(Ue, We, X[4], X[5]);
            X[6] = Uo + Wo;
            X[7] = Uo - Wo;
            h.fwd_regs(s0, s1, s2, s3, X[0], X[1], X[2], X[3]);
        }
    }
    __device__ __forceinline__ void inv(const V (&X)[NS], V (&x)[NS]) const
    {
        V Ue, We;
        h.join(X[4], X[5], Ue, We);
        const V Uo = X[6] + X[7], Wo = X[6] - X[7];
        V a = V(T(0)), b = V(T(0)), p = V(T(0)), q = V(T(0));
        block2<T>(h.C2T, Ue, a, h.C4, Uo, b);
        block2<T>(h.S2T, We, q, S4, Wo, p);
        const V A0 = a + b, A1 = a - b, B0 = p + q, B1 = p - q;
        V s0, s1, s2, s3;
        h.inv_regs(X[0], X[1], X[2], X[3], s0, s1, s2, s3);
        const V d0 = fma4<T>(A0, rc0, -(B0 * rs0)), d2 = fma4<T>(B0, rc0, A0 * rs0);
        const V d1 = fma4<T>(A1, rc1, -(B1 * rs1)), d3 = fma4<T>(B1, rc1, A1 * rs1);
        x[0] = s0 + d0;
        x[4] = s0 - d0;
        x[1] = s1 + d1;
        x[5] = s1 - d1;
        x[2] = s2 + d2;
        x[6] = s2 - d2;
        x[3] = s3 + d3;
        x[7] = s3 - d3;
    }
    __host__ __device__ static constexpr bool desc(int hb)
    {
        return (hb & 4) ? !Line64<T>::desc(hb & 3) : Line64<T>::desc(hb);
    }
    __host__ __device__ static constexpr int off(int hb)
    {
        return (hb & 4) ? 127 - Line64<T>::off(hb & 3) : Line64<T>::off(hb);
    }
    __host__ __device__ static constexpr int mode(int hb, int lab)
    {
        return hb < 4    ? 2 * Line64<T>::mode(hb, lab)
               : hb == 4 ? 8 * lab + 1
               : hb == 5 ? (lab == 0 ? 127 : 8 * lab - 1)
               : hb == 6 ? 8 * lab + 5
                         : 8 * lab + 3;
    }
};

// ------------------------------------------------- any n <= 32 NB, n >= 2
// One fold, then dense products of NB x NB blocks: positions j < ceil(n/2) and
// their mirrors, modes 2m and 2m + 1.  Constant blocks per n in operand order
// (k_mm_dense_const): [even | even transposed | odd][b'][b][lane][4]; in
// registers where they fit (kHeld), else read at each use (L1).
template <typename T, int NB>
struct LineDense {
    using V = Vec4<T>;
    static constexpr int N = 32 * NB, NS = 2 * NB;        // padded side
    static constexpr bool kRagged = true, kShort = false;
    static constexpr bool kHeld = NB == 1;
    static constexpr int kMats = 3 * NB * NB;
    V held[kHeld ? kMats : 1];
    __amdgpu_buffer_rsrc_t cst;
    unsigned at;
    __device__ __forceinline__ void init(const T *c, int lane)
    {
        cst = make_rsrc(c, kMats * 256 * sizeof(T));
        at = 4 * lane * sizeof(T);
        if constexpr (kHeld) {
#pragma unroll
            for (int k = 0; k < kMats; ++k) held[k] = read(k);
        }
    }
    // one uniform base and an immediate per block (a 64-bit address for each would be kept in scalars)
    __device__ __forceinline__ V read(int k) const
    {
        using U4 = __attribute__((ext_vector_type(4))) unsigned;
        const int bytes = k * 256 * (int)sizeof(T), so = bytes & ~4095, im = bytes & 4095;
        if constexpr (sizeof(T) == 4) {
            return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(cst, at + im, so, 0));
        } else {
            struct {
                U4 a, b;
            } r{__builtin_amdgcn_raw_buffer_load_b128(cst, at + im, so, 0),
                __builtin_amdgcn_raw_buffer_load_b128(cst, at + im + 16, so, 0)};
            return __builtin_bit_cast(V, r);
        }
    }
    __device__ __forceinline__ V mat(int m, int bo, int bi) const
    {
        const int k = (m * NB + bo) * NB + bi;
        if constexpr (kHeld) return held[k];
        else return read(k);
    }
    // keeps the reads of a later output block from being issued early, all at once
    __device__ __forceinline__ static void fence()
    {
        if constexpr (NB >= 3) __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void fwd(const V (&x)[NS], V (&X)[NS]) const
    {
#pragma unroll
        for (int bo = 0; bo < NB; ++bo) {
            X[bo] = V(T(0));
            X[NB + bo] = V(T(0));
#pragma unroll
            for (int b = 0; b < NB; ++b)
                block2<T>(mat(0, bo, b), x[b] + x[NB + b], X[bo], mat(2, bo, b), x[b] - x[NB + b], X[NB + bo]);
            fence();
        }
    }
    __device__ __forceinline__ void inv(const V (&X)[NS], V (&x)[NS]) const
    {
#pragma unroll
        for (int bo = 0; bo < NB; ++bo) {
            V e = V(T(0)), o = V(T(0));
#pragma unroll
            for (int b = 0; b < NB; ++b) block2<T>(mat(1, bo, b), X[b], e, mat(2, bo, b), X[NB + b], o);
            x[bo] = e + o;
            x[NB + bo] = e - o;
            fence();
        }
    }
    __host__ __device__ static constexpr bool desc(int hb) { return hb >= NB; }
    // the mirrors' offset depends on n: n - 1 - 16 b
    __host__ __device__ static constexpr int off(int hb, int n) { return hb < NB ? 16 * hb : n - 1 - 16 * (hb - NB); }
    __host__ __device__ static constexpr bool valid(int hb, int lab, int n)
    {
        return hb < NB ? 16 * hb + lab < (n + 1) / 2 : 16 * (hb - NB) + lab < n / 2;
    }
    // whether all labels of a block are valid: with NB the least that holds n, all blocks but the last of either half
    __host__ __device__ static constexpr bool full(int hb) { return hb % NB < NB - 1; }
    // -1: no such mode
    __host__ __device__ static constexpr int mode(int hb, int lab, int n)
    {
        const int k = hb < NB ? 2 * (16 * hb + lab) : 2 * (16 * (hb - NB) + lab) + 1;
        return k < n ? k : -1;
    }
};

// n <= 16: the lines' slots 8 .. 15 of either half, and so every second tile of
// eight lines, are padding.  The transforms are the same, for half the lines.
template <typename T>
struct LineShort : LineDense<T, 1> {
    static constexpr bool kShort = true;
};

// Uniform access to the slot maps of both kinds of line.
template <typename Line>
__host__ __device__ constexpr bool slot_valid(int hb, int lab, int n)
{
    if constexpr (Line::kRagged) return Line::valid(hb, lab, n);
    else return true;
}
template <typename Line>
__host__ __device__ constexpr bool slot_full(int hb)
{
    if constexpr (Line::kRagged) return Line::full(hb);
    else return true;
}
template <typename Line>
__host__ __device__ constexpr int slot_off(int hb, int n)
{
    if constexpr (Line::kRagged) return Line::off(hb, n);
    else return Line::off(hb);
}
template <typename Line>
__host__ __device__ constexpr int slot_pos(int hb, int lab, int n)
{
    return Line::desc(hb) ? slot_off<Line>(hb, n) - lab : slot_off<Line>(hb, n) + lab;
}
template <typename Line>
__host__ __device__ constexpr int slot_mode(int hb, int lab, int n)
{
    if constexpr (Line::kRagged) return Line::mode(hb, lab, n);
    else return Line::mode(hb, lab);
}

}  // namespace cil
