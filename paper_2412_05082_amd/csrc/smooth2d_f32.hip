// Instantiations of the 2D smoother kernels (smooth2d_impl.h) in float.
#include "smooth2d_impl.h"

namespace c0ip {

template hipError_t launch_step2d<float>(int, int, const LevelCoef<float>&, const LevelEig<float>&, const float*, const float*,
                                      float*, float, hipStream_t, int, int64_t, const int*, int, const float*, int64_t);
template hipError_t launch_pre2d_ref<float>(int, int, const LevelCoef<float>&, const LevelEig<float>&, const float*, float*, float*, float,
                                     hipStream_t);
template hipError_t launch_patch2d<float>(int, int, const LevelEig<float>&, const float*, const float*, float*, float, hipStream_t,
                                       int, int64_t, const int*);

}  // namespace c0ip
