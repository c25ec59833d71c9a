// FP64 instances of the matrix-core stepper's launches and tables.
#include "stepper_mm_launch.hpp"

namespace cil {

template int mm_make_tables<double>(int, const TabSpec *, int, double, double *, hipStream_t);
template int mm_make_consts<double>(int, double *, hipStream_t);
template int launch_mm<double>(int, int, int, const DevSolve *, const int *, double *, const double *, const double *,
                          const double *, int, double, const PersistArgs &, hipStream_t);

}  // namespace cil
