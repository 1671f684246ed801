// Launchers of the gfx950 kernels (internal to libc0ip; plain pointers).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace c0ip {

// Coefficient tables of one level's 1D M, L, B (row classes, see setup.h).
template <typename T>
struct LevelCoef {
  const T* tab = nullptr;  // [3][nclass][4k+1]
  int nclass = 0, left = 0, right0 = 0, periodic = 0;
  // With the default penalty: the same table scaled to h = 1 (M / h, L h,
  // B h^3), whose periodic rows are the compile-time reference rows, and
  // 1/h; ref == nullptr otherwise.
  const T* ref = nullptr;
  T hinv = 0;
};

// Fast-diagonalisation data of one level: Q[4][n*n], lam[4][n].
template <typename T>
struct LevelEig {
  const T* Q = nullptr;
  const T* lam = nullptr;
};

// y = A x, or y = b - A x when b != nullptr (boundary entries of y are 0).
// Tin = type of x, T = compute/output type.
template <typename Tin, typename T>
hipError_t launch_apply(int dim, int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y,
                        hipStream_t s);

// x_out = x_in + omega * sum_v R_v^T A~_v^{-1} R_v r  (x_in == nullptr: 0).
template <typename T>
hipError_t launch_patch_smooth(int dim, int k, int N, const LevelEig<T>& e, const T* r, const T* x_in,
                               T* x_out, T omega, hipStream_t s);

// Grid transfers (tensor-product 1D embedding, compile-time table): bc = P^T rf;
// xf += P ec.
template <typename T>
hipError_t launch_restrict(int dim, int k, int Nc, const T* rf, T* bc, hipStream_t s);
template <typename T>
hipError_t launch_prolong_add(int dim, int k, int Nc, const T* ec, T* xf, hipStream_t s);
template <typename T>
hipError_t launch_restrict3d(int k, int Nc, const T* rf, T* bc, hipStream_t s);
template <typename T>
hipError_t launch_prolong3d(int k, int Nc, const T* ec, T* xf, hipStream_t s);

// Level-0 solve: x = A0^{-1} b on the (2k-1)^dim interior nodes (float64);
// batched over nsys systems zs apart, skipping those with active[z] == 0.
template <typename T>
hipError_t launch_coarse(int dim, int k, const double* Ainv, const T* b, T* x, hipStream_t s, int nsys = 1,
                         int64_t zs = 0, const int* active = nullptr);

// Vector kernels (n = length).
template <typename Ta, typename Tb>
hipError_t launch_cast(int64_t n, const Ta* a, Tb* b, hipStream_t s);
hipError_t launch_fill(int64_t n, double v, double* a, hipStream_t s);
template <typename T>
hipError_t launch_fill_t(int64_t n, T v, T* a, hipStream_t s);
// partial[j * nblk + blk] = partial sum of V_j . w (j < m), nblk blocks.
hipError_t launch_multidot(int64_t n, int m, const double* V, int64_t ldv, const double* w, double* partial,
                           int nblk, hipStream_t s);
// out[j] = sum_b partial[j * nblk + b] (+ out_add[j] if accumulate)
hipError_t launch_reduce_partials(int m, int nblk, const double* partial, double* out, int accumulate,
                                  hipStream_t s);
// v = w / *nrm (nrm = device pointer to a squared norm: v = w / sqrt(*nrm))
hipError_t launch_normalize(int64_t n, const double* w, const double* nrm2, double* v, hipStream_t s);
// x += sum_j y[j] Z_j  (Z of type Tz)
template <typename Tz>
hipError_t launch_update_solution(int64_t n, int m, const Tz* Z, int64_t ldz, const double* y, double* x,
                                  hipStream_t s);

int multidot_blocks(int64_t n);

// Arnoldi step with delayed re-orthogonalisation (see kernels_common.hip).
// dots: partial[(2j+3) * nblk]; reduce_coef: d[2j+3] and coef[2j+5];
// update: V_j = (u - V s)/alpha into vout, u <- w - V f - (h_v/alpha) u.
int arnoldi_blocks(int64_t n);
hipError_t launch_arnoldi_dots(int64_t n, int j, const double* V, int64_t ldv, const double* u, const double* w,
                               double* partial, int nblk, hipStream_t s);
// d[row] = sum of partial row (2j+3 rows), then coef from d (2j+5 values);
// host: NULL or device-visible pinned memory that receives d at [0, 2j+3)
// and coef at [hoff, hoff + 2j+5), readable once the launches have completed.
hipError_t launch_arnoldi_reduce_coef(int j, int nblk, const double* partial, double* d, double* coef,
                                      double* host, int hoff, hipStream_t s);
// u32: NULL, or receives (float) of the new u (the next float32 V-cycle's input).
hipError_t launch_arnoldi_update(int64_t n, int j, const double* V, int64_t ldv, double* u, const double* w,
                                 const double* coef, double* vout, hipStream_t s, float* u32 = nullptr);

// Per-dimension operator and smoother launchers (k dispatched at run time).
// Batched forms (2D): nsys systems whose vectors are zs elements apart
// (fine / coarse strides zf / zc for the transfers); nsys = 1 for one.
// xc: NULL, or (one system) receives a copy of x, written from the staged
// tiles (saves a separate copy where x is needed again).
template <typename Tin, typename T>
hipError_t launch_apply2d(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s,
                          int nsys = 1, int64_t zs = 0, const int* active = nullptr, Tin* xc = nullptr);
// The same for the default penalty (c.ref set): compile-time coefficients.
template <typename Tin, typename T>
hipError_t launch_apply2d_ref(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s,
                              int nsys, int64_t zs, const int* active, Tin* xc);
template <typename T>
hipError_t launch_patch2d(int k, int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega,
                          hipStream_t s, int nsys = 1, int64_t zs = 0, const int* active = nullptr);
// xout += omega * sum_v R_v^T A~_v^{-1} R_v r with floating-point atomics
// (xout initialised by the caller; each patch solved once).
template <typename T>
hipError_t launch_patch2d_atomic(int k, int N, const LevelEig<T>& e, const T* r, T* xout, T omega, hipStream_t s);
// One colour of the coloured multiplicative smoother (2D, 8 colours):
// One colour of the 2D multiplicative smoother, in place on x:
// x += omega * sum over the colour's patches of R_v^T A~_v^{-1} R_v r.  With
// r == nullptr the launch forms r = b - A x on each patch's rows in LDS,
// from x as it is before the launch (the colour's patches are disjoint and
// A-orthogonal, and none reads the nodes another one writes); else r is
// read (a residual computed beforehand, or b when x is 0).
template <typename T>
hipError_t launch_mvs2d_colour(int k, int N, int colour, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b,
                               const T* r, T* x, T omega, hipStream_t s);
// The same with exact local solves (dense inverses Aex, layout as in exact.h).
template <typename T>
hipError_t launch_mvs2d_colour_exact(int k, int N, int colour, const LevelCoef<T>& c, const T* Aex, const T* b,
                                     const T* r, T* x, T omega, hipStream_t s);
// Both for the default penalty (c.ref set): fast diagonalisation with Q and
// lam, or exact local solves when Aex is given.
template <typename T>
hipError_t launch_mvs2d_colour_ref(int k, int N, int colour, const LevelCoef<T>& c, const T* Q, const T* lam,
                                   const T* Aex, const T* b, const T* r, T* x, T omega, hipStream_t s);
// One fused smoothing step S(x, b) (residual in LDS; x_out must not alias x).
// variant: tile-size variant (0 = default; below avs2d_variants(k)).  With ec:
// the step starts from x + P ec instead (ec: coarse vector of the level
// below, zc apart between systems; ptab: the embedding table).
template <typename T>
hipError_t launch_avs2d(int k, int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* x, const T* b, T* xout,
                        T omega, hipStream_t s, int nsys = 1, int64_t zs = 0, const int* active = nullptr,
                        int variant = 0, const T* ec = nullptr, const T* ptab = nullptr, int64_t zc = 0);
int avs2d_variants(int k);
// The same for the default penalty (c.ref set).
template <typename T>
hipError_t launch_step2d(int k, int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* x, const T* b, T* xout,
                         T omega, hipStream_t s, int nsys, int64_t zs, const int* active, int variant, const T* ec,
                         int64_t zc);
// x1 = S(0, b) and r = b - A x1 in one launch (default penalty k <= 5, others
// k <= 3, else hipErrorNotSupported).  It recomputes the solves of a two-cell
// halo, which pays only where launches and latency dominate: on levels up to
// pre2d_max_n(k, element size, default penalty) cells per direction (0:
// none).  Measured, fused against two launches, default penalty: Q3 128^2
// float32 7.1 against 9.4 us, 256^2 17.4 against 12.6; Q4 128^2 float64 14.3
// against 15, 64^2 8.1 against 10; Q6 64^2 float64 22.4 against 16.5.  Others,
// a whole V-cycle without the tail: float64 Q2 64^2 179 against 187, 128^2 218
// against 230; Q3 64^2 188 against 191, 128^2 235 against 234; float32 Q2
// 128^2 201 against 212, Q3 128^2 216 against 218.
inline int pre2d_max_n(int k, int elem_size, bool ref) {
  if (!ref) return k == 2 ? 128 : k == 3 ? (elem_size == 4 ? 128 : 64) : 0;
  return k <= 3 ? 128 : k == 4 ? (elem_size == 4 ? 128 : 64) : k == 5 ? 64 : 0;
}
template <typename T>
hipError_t launch_pre2d(int k, int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b, T* x1, T* r, T omega,
                        hipStream_t s);
// The same for the default penalty (c.ref set).
template <typename T>
hipError_t launch_pre2d_ref(int k, int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b, T* x1, T* r,
                            T omega, hipStream_t s);
template <typename T>
hipError_t launch_restrict2d(int k, int Nc, const T* rf, T* bc, hipStream_t s, int nsys = 1,
                             int64_t zf = 0, int64_t zc = 0, const int* active = nullptr);
// xf = xin + P ec (xin may equal xf)
template <typename T>
hipError_t launch_prolong2d(int k, int Nc, const T* ec, const T* xin, T* xf, hipStream_t s,
                            int nsys = 1, int64_t zc = 0, int64_t zf = 0, const int* active = nullptr);
template <typename Tin, typename T>
hipError_t launch_apply3d(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s);
// The same on boxes of cells (default penalty; any k).
template <typename Tin, typename T>
hipError_t launch_apply3d_box(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s);
// z-streaming operator with per-lane band loops (any k; used for other penalties).
template <typename Tin, typename T>
hipError_t launch_apply3d_wide(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s);
template <typename T>
hipError_t launch_patch3d(int k, int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega,
                          hipStream_t s);
// The same for k >= 4, on boxes of cells.
template <typename T>
hipError_t launch_patch3d_box(int k, int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega,
                              hipStream_t s);

// Lowest levels 0..LT of the 2D V-cycle in one launch, one workgroup per
// system, every vector in LDS (vtail.hip).  Tables as on the tiled path.
constexpr int kTailMaxLevels = 5;
template <typename T>
struct TailParams {
  int LT = 0;  // top level of the tail
  int nclass[kTailMaxLevels] = {}, left[kTailMaxLevels] = {}, right0[kTailMaxLevels] = {},
      periodic[kTailMaxLevels] = {};
  const T* tab[kTailMaxLevels] = {};
  const T* Q[kTailMaxLevels] = {};
  const T* lam[kTailMaxLevels] = {};
  const T* ptab = nullptr;       // embedding table [2][k][k+1]
  const double* Ainv = nullptr;  // level-0 inverse (coarse_mode 0)
  T omega = 0;
  int pre = 1, post = 1, coarse_mode = 0;
  bool ref = false;  // compile-time coefficients (vtail_ref.hip; default penalty), else tables (vtail.hip)
};
// Per-level slot buffers: system s exists on level l iff s < nA[l]; its
// vectors start at b[l] + s * stride[l] (x likewise).  A system's tail
// starts at its highest level <= LT: b there is read, x there is written.
template <typename T>
struct TailIO {
  const T* b[kTailMaxLevels] = {};
  T* x[kTailMaxLevels] = {};
  int64_t stride[kTailMaxLevels] = {};
  int nA[kTailMaxLevels] = {};
  const int* active = nullptr;
};
// LDS bytes of the tail kernel for degree k up to level LT (nclass per level,
// or NULL for the default penalty's kernel).
int tail_bytes(int k, int LT, const int* nclass, int elem_size);
int tail_ref_bytes(int k, int LT, int elem_size);
// Whether the tail with compile-time coefficients is the faster one for the
// default penalty (levels 0..LT, steps = pre + post).  Not in float64 on the
// smallest meshes: there a wave's items are few and long, and each of their
// coefficients takes two scalar moves, where the tables' kernel spreads an
// output to a lane.  Per smoothing step and level 0.4 to 1.6 us more; what the
// transfers and the coarse solve save makes up for it in one step each way at
// degrees 2 and 4.  V-cycle in us, compile-time against tables, 1+1 and 2+2
// steps: Q3 4^2 18.5 and 17.5, 29.9 and 25.0; 8^2 34.8 and 31.7, 59.3 and
// 49.9; 16^2 61.2 and 65.2, 109 and 112; Q2 8^2 22.7 and 24.0, 37.1 and 35.7;
// 16^2 35.7 and 38.3, 60.8 and 60.9; Q4 4^2 23.1 and 24.5, 37.7 and 35.7; 8^2
// 45 and 59, 78 and 90.
inline bool tail_ref_better(int k, int LT, int elem_size, int steps) {
  if (elem_size == 4) return true;
  if (k == 3) return LT > 2;
  return steps < 4 || LT > (k == 2 ? 3 : 1);
}
// Largest LDS a workgroup may use on the current device.
int tail_lds_limit();
// Allow the tail kernel of degree k `bytes` of dynamic LDS (before launch or capture).
template <typename T>
hipError_t configure_vtail(int k, int bytes);
template <typename T>
hipError_t configure_vtail_ref(int k, int bytes);
template <typename T>
hipError_t launch_vtail_ref(int k, const TailParams<T>& P, const TailIO<T>& io, int nsys, hipStream_t s);
template <typename T>
hipError_t launch_vtail(int k, const TailParams<T>& P, const TailIO<T>& io, int nsys, hipStream_t s);

#define C0IP_DISPATCH_K(k, CALL)          \
  switch (k) {                            \
    case 2: return CALL(2);               \
    case 3: return CALL(3);               \
    case 4: return CALL(4);               \
    case 5: return CALL(5);               \
    case 6: return CALL(6);               \
    case 7: return CALL(7);               \
    default: return hipErrorInvalidValue; \
  }

}  // namespace c0ip
