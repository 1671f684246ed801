// One colour of the coloured multiplicative smoother on a 3D mesh (internal
// to libc0ip; plain pointers).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace c0ip {

// Lattice of a colour along one axis (a, b, cc of the numbering in mvs3d.hip).
struct Lat {
  int lo, hi;  // lattice index range along one axis
};

__host__ __device__ inline Lat lat(int N, int par) { return {par == 0 ? 1 : 0, (N - 1 - par) / 2}; }

__host__ __device__ inline int row_count(Lat a, int b, int par) {
  const int af = a.lo + (((par - a.lo - b) % 2) + 2) % 2;
  return af <= a.hi ? (a.hi - af) / 2 + 1 : 0;
}

// The same for the default penalty and k <= 4 (mvs3d_ref.hip); r == nullptr:
// the launch forms r = b - A x on the patches itself.
template <typename T>
hipError_t launch_mvs3d_colour_ref(int k, int N, int colour, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b,
                                   const T* r, T* x, T omega, hipStream_t s);

// x += omega * sum over colour c's patches of R_v^T A~_v^{-1} R_v r, in
// place (16 colours; the colour's patches are disjoint and A-orthogonal).
template <typename T>
hipError_t launch_mvs3d_colour(int k, int N, int colour, const LevelEig<T>& e, const T* r, T* x, T omega,
                               hipStream_t s);

}  // namespace c0ip
