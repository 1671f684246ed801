// The 2D matrix-free operator for the default penalty (Sec. 4, eq.
// c0iptensorvp used on the whole Cartesian mesh): y = A x or y = b - A x,
// one workgroup per tile of whole cells (tile2d.h).
#include "kernels.h"
#include "tile2d.h"

namespace c0ip {
namespace {

using tile2::Op;

// Three phases (stage, x pass, y pass).  2D Q3 64^2 float32 11.4 -> 3.6 us:
// what went is the latency of six passes, each waiting for its coefficients
// in scalar registers, and the second, per-lane product of boundary rows.
// Large meshes are bound by vector issue: in float64 two scalar moves per
// coefficient ride along (Q3 512^2 float64 18.8 -> 17.7 us, float32 14.5 ->
// 9.7, Q2 512^2 float64 16.3 -> 8.3, Q4 512^2 float64 39 -> 30).
template <typename Tin, typename T, class G, bool RES>
__global__ __launch_bounds__(G::NTH) void apply2d_ref_kernel(const Tin* __restrict__ x, const T* __restrict__ b,
                                                             T* __restrict__ y, int N, int n1, T scale, int64_t zs,
                                                             const int* __restrict__ active, int tx, int total,
                                                             Tin* __restrict__ xc) {
  if (active && !active[blockIdx.z]) return;
  constexpr int K = G::K;
  const int tile = tile2::xcd_order(blockIdx.x, total), bx = tile % tx, by = tile / tx;
  const int cx0 = bx * G::TXC, cy0 = by * G::TYC, x0 = cx0 * K, y0 = cy0 * K, NK = n1 - 1;
  x += blockIdx.z * zs;
  y += blockIdx.z * zs;
  if (RES) b += blockIdx.z * zs;
  __shared__ T sX[G::SZX];
  __shared__ T sT[G::SZT];
  tile2::StageX<Tin, T, G> st;
  st.load(x, x0 - G::H, y0 - G::H, n1);
  // b of the outputs (residual form), loaded now to overlap the passes
  T bv[RES ? G::NI : 1][K];
  if constexpr (RES) {
    const tile2::Rows<T> bb(b, n1, max(y0, 1), min(y0 + G::TY, NK) - 1);
#pragma unroll
    for (int q = 0; q < G::NI; ++q) {
      const int it = threadIdx.x + q * G::NTH, cy = it / G::TX, l = it - cy * G::TX, gx = x0 + l;
      const bool on = it < G::NY && gx >= 1 && gx < NK;
#pragma unroll
      for (int p = 0; p < K; ++p) bv[q][p] = bb.load(on ? bb.off(y0 + cy * K + p, gx) : tile2::kOff);
    }
  }
  st.store(sX);
  // the last node row and column (boundary) belong to the last tiles
  if (cx0 + G::TXC >= N) {
    for (int e = threadIdx.x; e < G::TY; e += G::NTH)
      if (y0 + e < NK) {
        y[(size_t)(y0 + e) * n1 + NK] = T(0);
        if (xc) xc[(size_t)(y0 + e) * n1 + NK] = Tin(0);
      }
  }
  if (cy0 + G::TYC >= N) {
    for (int e = threadIdx.x; e <= G::TX; e += G::NTH)
      if (x0 + e < NK || (x0 + e == NK && cx0 + G::TXC >= N)) {
        y[(size_t)NK * n1 + x0 + e] = T(0);
        if (xc) xc[(size_t)NK * n1 + x0 + e] = Tin(0);
      }
  }
  __syncthreads();
  tile2::op_x<T, G>(sX, sT, cx0, N);
  __syncthreads();
  const int rhi = min(y0 + G::TY, NK) - 1;
  const tile2::Rows<T> yb(y, n1, y0, rhi);
  const tile2::Rows<Tin> xb(xc ? xc : x, n1, y0, xc ? rhi : y0 - 1);
#pragma unroll
  for (int q = 0; q < G::NI; ++q) {
    const int it = threadIdx.x + q * G::NTH;
    if (G::NY % G::NTH != 0 && it >= G::NY) break;
    const int cy = it / G::TX, l = it - cy * G::TX, gx = x0 + l;
    T acc[K];
    tile2::op_y<T, G>(sT, acc, l, cy, cy0 + cy, N);
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int gy = y0 + cy * K + p;
      const T a = gx == 0 || gy == 0 ? T(0) : scale * acc[p];
      yb.store(gx < NK ? yb.off(gy, gx) : tile2::kOff, RES ? bv[q][p] - a : a);
      if (xc)  // exact: T holds every Tin
        xb.store(gx < NK ? xb.off(gy, gx) : tile2::kOff, (Tin)sX[(cy * K + p + G::H) * G::RXP + l + G::H]);
    }
  }
}

template <typename Tin, typename T, class G>
hipError_t apply2d_ref_g(int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s, int nsys,
                         int64_t zs, const int* active, Tin* xc) {
  const int n1 = G::K * N + 1, tx = (N + G::TXC - 1) / G::TXC, total = tx * ((N + G::TYC - 1) / G::TYC);
  const dim3 grid(total, 1, nsys);
  const T scale = c.hinv * c.hinv;
  if (b)
    apply2d_ref_kernel<Tin, T, G, true><<<grid, G::NTH, 0, s>>>(x, b, y, N, n1, scale, zs, active, tx, total, xc);
  else
    apply2d_ref_kernel<Tin, T, G, false><<<grid, G::NTH, 0, s>>>(x, b, y, N, n1, scale, zs, active, tx, total, xc);
  return hipGetLastError();
}

// Tiles per degree (and type, where that differs), by sweeps at 256^2 and
// 512^2 cells.  Float64 rounds fill the chip with small tiles; float32 at
// k = 2, 3 gains from the smaller halo of 16 x 16 cells (Q3 512^2 float32:
// 9.7 us against 11.0 with 8 x 8; float64: 20 against 17.7).
template <typename T, int K> struct Cfg;
template <typename T> struct Cfg<T, 2> { using G = Op<2, 16, 16, 512, 2>; };
template <> struct Cfg<float, 3> { using G = Op<3, 16, 16, 512, 2>; };
template <> struct Cfg<double, 3> { using G = Op<3, 8, 8, 192, 2>; };
template <typename T> struct Cfg<T, 4> { using G = Op<4, 8, 8, 256, 2>; };
template <typename T> struct Cfg<T, 5> { using G = Op<5, 4, 8, 256, 1>; };
template <typename T> struct Cfg<T, 6> { using G = Op<6, 8, 4, 512, 1>; };
template <typename T> struct Cfg<T, 7> { using G = Op<7, 4, 4, 256, 1>; };

template <typename Tin, typename T, int K>
hipError_t apply2d_ref_k(int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s, int nsys,
                         int64_t zs, const int* active, Tin* xc) {
  using G = typename Cfg<T, K>::G;
  // Meshes with fewer tiles than compute units are bound by the latency of
  // one workgroup: 4 x 4 cells over four waves (Q3 64^2: 3.6 us against 4.1
  // with 8 x 8 cells and 4.5 with one wave)
  const int64_t big = (int64_t)((N + G::TXC - 1) / G::TXC) * ((N + G::TYC - 1) / G::TYC) * nsys;
  if (big < 256) return apply2d_ref_g<Tin, T, Op<K, 4, 4, 256, 1>>(N, c, x, b, y, s, nsys, zs, active, xc);
  return apply2d_ref_g<Tin, T, G>(N, c, x, b, y, s, nsys, zs, active, xc);
}


}  // namespace

template <typename Tin, typename T>
hipError_t launch_apply2d_ref(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s,
                              int nsys, int64_t zs, const int* active, Tin* xc) {
  if (xc && nsys != 1) return hipErrorInvalidValue;
#define CALL(K) apply2d_ref_k<Tin, T, K>(N, c, x, b, y, s, nsys, zs, active, xc)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

template hipError_t launch_apply2d_ref<double, double>(int, int, const LevelCoef<double>&, const double*,
                                                       const double*, double*, hipStream_t, int, int64_t, const int*,
                                                       double*);
template hipError_t launch_apply2d_ref<float, double>(int, int, const LevelCoef<double>&, const float*,
                                                      const double*, double*, hipStream_t, int, int64_t, const int*,
                                                      float*);
template hipError_t launch_apply2d_ref<float, float>(int, int, const LevelCoef<float>&, const float*, const float*,
                                                     float*, hipStream_t, int, int64_t, const int*, float*);

}  // namespace c0ip
