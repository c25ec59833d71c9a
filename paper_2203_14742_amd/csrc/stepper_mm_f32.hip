// FP32 instances of the matrix-core stepper's launches and tables.
#include "stepper_mm_launch.hpp"

namespace cil {

template int mm_make_tables<float>(int, const TabSpec *, int, double, float *, hipStream_t);
template int mm_make_consts<float>(int, float *, hipStream_t);
template int launch_mm<float>(int, int, int, const DevSolve *, const int *, float *, const float *, const float *,
                          const float *, int, double, const PersistArgs &, hipStream_t);

}  // namespace cil
