// Instantiations of the 2D smoother kernels (smooth2d_impl.h) in double.
#include "smooth2d_impl.h"

namespace c0ip {

template hipError_t launch_step2d<double>(int, int, const LevelCoef<double>&, const LevelEig<double>&, const double*, const double*,
                                      double*, double, hipStream_t, int, int64_t, const int*, int, const double*, int64_t);
template hipError_t launch_pre2d_ref<double>(int, int, const LevelCoef<double>&, const LevelEig<double>&, const double*, double*, double*, double,
                                     hipStream_t);
template hipError_t launch_patch2d<double>(int, int, const LevelEig<double>&, const double*, const double*, double*, double, hipStream_t,
                                       int, int64_t, const int*);

}  // namespace c0ip
