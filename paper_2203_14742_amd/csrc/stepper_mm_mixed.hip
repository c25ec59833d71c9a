// Mixed-precision instances of the matrix-core stepper: FP32 steps, then from
// the FP32 floor to the tolerance either the refinement form or FP64 steps.
#include "stepper_mm.hpp"

namespace cil {

namespace {

template <typename LineF, typename LineD, int TPW, int WPE, bool RF>
void launch_mixed(int model, int nl, const DevSolve *S, const int *list, float *state, double *state64,
                  const float *tab32, const double *tab64, double dt, const PersistArgs &pa32, const PersistArgs &pa64,
                  long long *switch_step, int mode, hipStream_t st)
{
    constexpr int threads = MmShape<float, LineF, TPW>::THREADS;
    dispatch_model(model, [&](auto MD) {
        hipLaunchKernelGGL((k_mm_mixed<decltype(MD)::value, LineF, LineD, TPW, WPE, RF>), dim3(nl), dim3(threads), 0,
                           st, S, list, state, state64, tab32, tab64, dt, pa32, pa64, switch_step, mode);
    });
}

}  // namespace

int launch_mm_mixed(int n, int nl, const DevSolve *S, const int *list, float *state, double *state64,
                    const float *tab32, const double *tab64, int model, double dt, const PersistArgs &pa32,
                    const PersistArgs &pa64, long long *switch_step, int refine, int mode, hipStream_t st)
{
    auto go = [&](auto lf, auto ld, auto tpw, auto wpe, auto rf) {
        launch_mixed<decltype(lf), decltype(ld), decltype(tpw)::value, decltype(wpe)::value, decltype(rf)::value>(
            model, nl, S, list, state, state64, tab32, tab64, dt, pa32, pa64, switch_step, mode, st);
    };
    using std::integral_constant;
    using I1 = integral_constant<int, 1>;
    using I2 = integral_constant<int, 2>;
    using I4 = integral_constant<int, 4>;
    // FP64 steps at 64 take two tiles a wavefront: four wavefronts of 256
    // registers, so that two solves still share a CU
    if (n == 32 && refine) go(Line32<float>{}, Line32<double>{}, I1{}, I4{}, std::true_type{});
    else if (n == 32) go(Line32<float>{}, Line32<double>{}, I1{}, I4{}, std::false_type{});
    else if (n == 64 && refine) go(Line64<float>{}, Line64<double>{}, I1{}, I4{}, std::true_type{});
    else if (n == 64) go(Line64<float>{}, Line64<double>{}, I2{}, I2{}, std::false_type{});
    else return CIL_EUNSUPPORTED;
    return CIL_OK;
}

}  // namespace cil
