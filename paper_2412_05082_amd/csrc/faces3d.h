// The boundary faces that the 3D operators' tiles do not own.
#pragma once

#include <hip/hip_runtime.h>

namespace c0ip {
namespace {

// Zeros on the faces x = kN, y = kN, z = kN (boundary nodes that no tile
// owns): face element f of 3 n1^2, 16 per thread.
template <typename T, int NTH>
__device__ __forceinline__ void zero_faces(T* __restrict__ y, int n1, int fb) {
  const int NK = n1 - 1;
  const int64_t nf = (int64_t)n1 * n1;
  for (int q = 0; q < 16; ++q) {
    const int64_t f = ((int64_t)fb * 16 + q) * NTH + threadIdx.x;
    if (f >= 3 * nf) return;
    const int face = (int)(f / nf);
    const int64_t rem = f - face * nf;
    const int u = (int)(rem % n1), w = (int)(rem / n1);
    const int gx = face == 0 ? NK : u, gy = face == 0 ? u : (face == 1 ? NK : w), gz = face == 2 ? NK : w;
    y[((size_t)gz * n1 + gy) * n1 + gx] = T(0);
  }
}
template <int NTH>
inline int face_blocks(int n1) {
  return (int)((3 * (int64_t)n1 * n1 + 16 * NTH - 1) / (16 * NTH));
}

}  // namespace
}  // namespace c0ip
