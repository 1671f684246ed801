#pragma once
// 2D additive vertex-patch smoother for the default penalty, owner computes
// (Sec. 3; local solver of eq. localsolverbila inverted by eq. inverse):
//   x_out = x + omega * sum_v R_v^T (Q_y (x) Q_x) D_v^{-1} (Q_y (x) Q_x)^T R_v (b - A x).
// A workgroup owns TC x TC cells and solves the (TC+1)^2 patches that touch
// them (neighbouring tiles solve shared patches twice instead of racing on
// writes), writing each owned DoF once (no atomics, deterministic).
//   step2d:  x_out = S(x, b), or S(x + P e, b) (first post-smoothing step);
//   pre2d:   x1 = S(0, b) and r = b - A x1 (first pre-smoothing step and the
//            residual after it);
//   patch2d: x_out = x_in + the local solves of a given residual.
// All three are built from the phases of tile2d.h: the residual on the tile
// extended by one cell stays in LDS.
#include "kernels.h"
#include "tile2d.h"

namespace c0ip {
namespace {

using tile2::Fd;
using tile2::kOff;
using tile2::Op;
using tile2::Rows;

constexpr int cmax(int a, int b) { return a > b ? a : b; }

// The interior eigenbasis through scalar registers when it fits 64 of them,
// else from LDS like the other variants.
template <typename T, int K>
constexpr bool kScalarQ = (2 * K - 1) * (2 * K - 1) * (int)sizeof(T) / 4 <= 64;

// Phases 3 and 4: R (row stride rp, first patch node) -> x modes -> y solves in sU.
template <typename T, class S>
__device__ __forceinline__ void patch_phases(const T* __restrict__ sR, int rp, T* __restrict__ sM,
                                             T* __restrict__ sU, const T* __restrict__ Qg, const T* __restrict__ sQ,
                                             const T* __restrict__ sLam, const T* __restrict__ sD, int cx0, int cy0,
                                             int N, bool interior) {
  const T* q0 = kScalarQ<T, S::K> ? Qg : sQ;
  if (interior)
    tile2::fd_x<T, S, true>(sR, rp, sM, q0, sQ, cx0, N);
  else
    tile2::fd_x<T, S, false>(sR, rp, sM, q0, sQ, cx0, N);
  __syncthreads();
  if (interior)
    tile2::fd_y<T, S, true>(sM, sU, q0, sQ, sLam, sD, cx0, cy0, N);
  else
    tile2::fd_y<T, S, false>(sM, sU, q0, sQ, sLam, sD, cx0, cy0, N);
  __syncthreads();
}

template <typename T, class S>
__device__ __forceinline__ void corrections(const T* __restrict__ sU, T (&a)[S::K], const T* __restrict__ Qg,
                                            const T* __restrict__ sQ, int oy, int c, int cx0, int N, bool interior) {
  const T* q0 = kScalarQ<T, S::K> ? Qg : sQ;
  if (interior)
    tile2::fd_out<T, S, true>(sU, a, q0, sQ, oy, c, cx0, N);
  else
    tile2::fd_out<T, S, false>(sU, a, q0, sQ, oy, c, cx0, N);
}

// Write the owned nodes (row oy, cell c of the tile): v[p] = x + omega a, 0 on the boundary.
template <typename T, class S>
__device__ __forceinline__ void write_owned(const Rows<T>& out, const T (&xv)[S::K], const T (&a)[S::K], T omega,
                                            int oy, int c, int cx0, int cy0, int N) {
  constexpr int K = S::K;
  const int gx = (cx0 + c) * K, gy = cy0 * K + oy;
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const bool bnd = gy == 0 || gx + p == 0;
    out.store(cx0 + c < N ? out.off(gy, gx + p) : kOff, bnd ? T(0) : xv[p] + omega * a[p]);
  }
}

// The last node row and column of the mesh (boundary) belong to the last tiles.
template <typename T, int OWN, int NTH>
__device__ __forceinline__ void zero_last(T* __restrict__ x, int gx0, int gy0, int n1) {
  const int NK = n1 - 1;
  if (gx0 + OWN >= NK) {
    for (int e = threadIdx.x; e < OWN; e += NTH)
      if (gy0 + e < NK) x[(size_t)(gy0 + e) * n1 + NK] = T(0);
  }
  if (gy0 + OWN >= NK) {
    for (int e = threadIdx.x; e <= OWN; e += NTH)
      if (gx0 + e < NK || (gx0 + e == NK && gx0 + OWN >= NK)) x[(size_t)NK * n1 + gx0 + e] = T(0);
  }
}

// ------------------------------------------------------------------ step2d
template <typename T, int K_, int TC_, int NTH_, int CW_, bool PRO>
struct StepCfg {
  using S = Fd<K_, TC_, NTH_>;
  using G = Op<K_, TC_ + 2, TC_ + 2, NTH_, CW_>;
  using PR = tile2::Prolong<T, G>;
  static constexpr int RP = G::TXP;  // residual rows: TY x TX nodes
  // region A: staged x, then the residual, then the y solves; region B: the
  // prolongation's scratch, the operator's x passes, then the x modes
  static constexpr int A = cmax(G::SZX, cmax(G::TY * RP, S::SZU));
  static constexpr int B = cmax(cmax(G::SZT, S::SZM), PRO ? PR::SZC + PR::SZP : 0);
  static constexpr int BYTES = (A + B + 5 * S::NN + 4 * S::n) * (int)sizeof(T);
};

// Small meshes are bound by the latency of the phases (5 barriers, 7 with
// the prolongation, in place of 11 and 13): Q3 64^2 float32 17.2 -> 5.4 us,
// Q4 64^2 float64 28.2 -> 7.4.  Large ones by vector issue and LDS: Q3 512^2
// float32 35.3 -> 25.0 us, float64 57 -> 44.6; Q6 128^2 float64 84 -> 51.
template <typename T, class C, bool PRO>
__global__ __launch_bounds__(C::S::NTH) void step2d_kernel(const T* __restrict__ x, const T* __restrict__ b,
                                                           T* __restrict__ xout, int N, int n1, T scale,
                                                           const T* __restrict__ Qg, const T* __restrict__ lamg,
                                                           T omega, int64_t zs, const int* __restrict__ active,
                                                           int tx, int total, const T* __restrict__ ec, int64_t zc) {
  using S = typename C::S;
  using G = typename C::G;
  constexpr int K = S::K, TC = S::TC, NTH = S::NTH;
  if (active && !active[blockIdx.z]) return;
  __shared__ T sA[C::A];
  __shared__ T sB[C::B];
  __shared__ T sQ[4 * S::NN];
  __shared__ T sLam[4 * S::n];
  __shared__ T sD[S::NN];
  const int tile = tile2::xcd_order(blockIdx.x, total), bx = tile % tx, by = tile / tx;
  x += blockIdx.z * zs;
  b += blockIdx.z * zs;
  xout += blockIdx.z * zs;
  if (PRO) ec += blockIdx.z * zc;
  const int cx0 = bx * TC, cy0 = by * TC, x0 = (cx0 - 1) * K, y0 = (cy0 - 1) * K, NK = n1 - 1;
  tile2::StageX<T, T, G> st;
  st.load(x, x0 - G::H, y0 - G::H, n1);
  typename C::PR pr;
  if constexpr (PRO) pr.load(ec, cx0 - 1, cy0 - 1, N);
  tile2::StageEig<T, S::n, NTH> eig;
  eig.load(Qg, lamg);
  // b on the residual tile, loaded now to overlap the passes
  T bv[G::NI][K];
  {
    const Rows<T> bb(b, n1, max(y0, 1), min(y0 + G::TY, NK) - 1);
#pragma unroll
    for (int q = 0; q < G::NI; ++q) {
      const int it = threadIdx.x + q * NTH, cy = it / G::TX, l = it - cy * G::TX, gx = x0 + l;
      const bool on = it < G::NY && gx >= 1 && gx < NK;
#pragma unroll
      for (int p = 0; p < K; ++p) bv[q][p] = bb.load(on ? bb.off(y0 + cy * K + p, gx) : kOff);
    }
  }
  st.store(sA);
  if constexpr (PRO) pr.store(sB);
  eig.store(sQ, sLam, sD);
  zero_last<T, S::OWN, NTH>(xout, cx0 * K, cy0 * K, n1);
  __syncthreads();
  if constexpr (PRO) {
    C::PR::along_x(sB, sB + C::PR::SZC);
    __syncthreads();
    C::PR::along_y(sB + C::PR::SZC, sA);
    __syncthreads();
  }
  tile2::op_x<T, G>(sA, sB, cx0 - 1, N);
  // x of this thread's outputs, before the residual takes the staged tile's place
  T xv[S::NO][K];
#pragma unroll
  for (int q = 0; q < S::NO; ++q) {
    const int it = threadIdx.x + q * NTH, oy = it / TC, c = it - oy * TC;
#pragma unroll
    for (int p = 0; p < K; ++p)
      xv[q][p] = it < S::OWN * TC ? sA[(oy + K + G::H) * G::RXP + (c + 1) * K + p + G::H] : T(0);
  }
  __syncthreads();
  // r = b - A x (0 on and outside the boundary)
#pragma unroll
  for (int q = 0; q < G::NI; ++q) {
    const int it = threadIdx.x + q * NTH;
    if (G::NY % NTH != 0 && it >= G::NY) break;
    const int cy = it / G::TX, l = it - cy * G::TX, gx = x0 + l;
    T acc[K];
    tile2::op_y<T, G>(sB, acc, l, cy, cy0 - 1 + cy, N);
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int gy = y0 + cy * K + p;
      const bool inner = gx >= 1 && gx < NK && gy >= 1 && gy < NK;
      sA[(cy * K + p) * C::RP + l] = inner ? bv[q][p] - scale * acc[p] : T(0);
    }
  }
  __syncthreads();
  const bool interior = cx0 >= 2 && cx0 + TC <= N - 2 && cy0 >= 2 && cy0 + TC <= N - 2;
  // the x modes are complete before the y solves overwrite the residual
  patch_phases<T, S>(sA + C::RP + 1, C::RP, sB, sA, Qg, sQ, sLam, sD, cx0, cy0, N, interior);
  const Rows<T> out(xout, n1, cy0 * K, min(cy0 * K + S::OWN, NK) - 1);
#pragma unroll
  for (int q = 0; q < S::NO; ++q) {
    const int it = threadIdx.x + q * NTH, oy = it / TC, c = it - oy * TC;
    if ((S::OWN * TC) % NTH != 0 && it >= S::OWN * TC) break;
    T a[K];
    corrections<T, S>(sA, a, Qg, sQ, oy, c, cx0, N, interior);
    write_owned<T, S>(out, xv[q], a, omega, oy, c, cx0, cy0, N);
  }
}

template <typename T, int K, int TC, int NTH, int CW>
hipError_t step2d_g(int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* x, const T* b, T* xout, T omega,
                    hipStream_t s, int nsys, int64_t zs, const int* active, const T* ec, int64_t zc) {
  const int n1 = K * N + 1, tx = (N + TC - 1) / TC;
  const dim3 grid(tx * tx, 1, nsys);
  const T scale = c.hinv * c.hinv;
  if (ec)
    step2d_kernel<T, StepCfg<T, K, TC, NTH, CW, true>, true><<<grid, NTH, 0, s>>>(
        x, b, xout, N, n1, scale, e.Q, e.lam, omega, zs, active, tx, tx * tx, ec, zc);
  else
    step2d_kernel<T, StepCfg<T, K, TC, NTH, CW, false>, false><<<grid, NTH, 0, s>>>(
        x, b, xout, N, n1, scale, e.Q, e.lam, omega, zs, active, tx, tx * tx, ec, zc);
  return hipGetLastError();
}

// ------------------------------------------------------------------- pre2d
// The residual on the tile needs x1 on the tile extended by two cells, so
// the workgroup solves every patch covering that region from b staged on
// three more cells; the redundant solves replace a launch and a round trip of
// x1 through memory.
template <typename T, int K_, int TC_, int NTH_, int CW_>
struct PreCfg {
  using G = Op<K_, TC_, TC_, NTH_, CW_>;
  using S = Fd<K_, TC_ + 4, NTH_>;
  static constexpr int BW = S::RS, BP = BW | 1;  // staged b
  // region A: b, then x1; region B: x modes, then the operator's x passes; U: y solves
  static constexpr int A = cmax(BW * BP, G::SZX), B = cmax(S::SZM, G::SZT);
  static constexpr int BYTES = (A + B + S::SZU + 5 * S::NN + 4 * S::n) * (int)sizeof(T);
};

// Bound by the latency of its phases: Q3 N <= 64 float32 14.4 -> 5.6 us, Q2
// 9.7 -> 4.7; it replaces 12.8 + 16.1 us in two launches for Q4 N <= 64
// float64 by 8.1.
template <typename T, class C>
__global__ __launch_bounds__(C::S::NTH) void pre2d_kernel(const T* __restrict__ b, T* __restrict__ x1out,
                                                          T* __restrict__ rout, int N, int n1, T scale,
                                                          const T* __restrict__ Qg, const T* __restrict__ lamg,
                                                          T omega, int64_t zs, int tx, int total) {
  using S = typename C::S;
  using G = typename C::G;
  constexpr int K = S::K, TC = G::TXC, NTH = S::NTH, EC = S::TC;
  __shared__ T sA[C::A];
  __shared__ T sB[C::B];
  __shared__ T sU[S::SZU];
  __shared__ T sQ[4 * S::NN];
  __shared__ T sLam[4 * S::n];
  __shared__ T sD[S::NN];
  const int tile = tile2::xcd_order(blockIdx.x, total), bx = tile % tx, by = tile / tx;
  b += blockIdx.z * zs;
  x1out += blockIdx.z * zs;
  rout += blockIdx.z * zs;
  const int cx0 = bx * TC, cy0 = by * TC, x0 = cx0 * K, y0 = cy0 * K, NK = n1 - 1;
  const int ex0 = cx0 - 2, ey0 = cy0 - 2;  // first cell of the x1 region
  tile2::Stage<T, T, C::BW, C::BW, C::BP, NTH> st;
  st.load(b, (ex0 - 1) * K + 1, (ey0 - 1) * K + 1, n1);
  tile2::StageEig<T, S::n, NTH> eig;
  eig.load(Qg, lamg);
  st.store(sA);
  eig.store(sQ, sLam, sD);
  zero_last<T, G::TX, NTH>(x1out, x0, y0, n1);
  zero_last<T, G::TX, NTH>(rout, x0, y0, n1);
  __syncthreads();
  const bool interior = ex0 >= 2 && ex0 + EC <= N - 2 && ey0 >= 2 && ey0 + EC <= N - 2;
  // b of the owned nodes, before x1 takes the staged tile's place
  T bv[G::NI][K];
#pragma unroll
  for (int q = 0; q < G::NI; ++q) {
    const int it = threadIdx.x + q * NTH, cy = it / G::TX, l = it - cy * G::TX;
#pragma unroll
    for (int p = 0; p < K; ++p)
      bv[q][p] = it < G::NY ? sA[(cy * K + p + 3 * K - 1) * C::BP + l + 3 * K - 1] : T(0);
  }
  patch_phases<T, S>(sA, C::BP, sB, sU, Qg, sQ, sLam, sD, ex0, ey0, N, interior);
  // x1 on the operator's staged region, 0 on and outside the boundary
  for (int it = threadIdx.x; it < S::OWN * EC; it += NTH) {
    const int oy = it / EC, c = it - oy * EC;
    T a[K];
    corrections<T, S>(sU, a, Qg, sQ, oy, c, ex0, N, interior);
    const int gy = ey0 * K + oy;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int gx = (ex0 + c) * K + p;
      sA[oy * G::RXP + c * K + p] = gx >= 1 && gx < NK && gy >= 1 && gy < NK ? omega * a[p] : T(0);
    }
  }
  __syncthreads();
  tile2::op_x<T, G>(sA, sB, cx0, N);
  __syncthreads();
  const int rhi = min(y0 + G::TY, NK) - 1;
  const Rows<T> xo(x1out, n1, y0, rhi), ro(rout, n1, y0, rhi);
#pragma unroll
  for (int q = 0; q < G::NI; ++q) {
    const int it = threadIdx.x + q * NTH;
    if (G::NY % NTH != 0 && it >= G::NY) break;
    const int cy = it / G::TX, l = it - cy * G::TX, gx = x0 + l;
    T acc[K];
    tile2::op_y<T, G>(sB, acc, l, cy, cy0 + cy, N);
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int gy = y0 + cy * K + p;
      const unsigned o = gx < NK ? xo.off(gy, gx) : kOff;
      xo.store(o, sA[(cy * K + p + G::H) * G::RXP + l + G::H]);
      ro.store(o, gx == 0 || gy == 0 ? T(0) : bv[q][p] - scale * acc[p]);
    }
  }
}

template <typename T, int K, int TC, int NTH, int CW>
hipError_t pre2d_g(int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b, T* x1, T* r, T omega,
                   hipStream_t s) {
  const int n1 = K * N + 1, tx = (N + TC - 1) / TC;
  pre2d_kernel<T, PreCfg<T, K, TC, NTH, CW>><<<tx * tx, NTH, 0, s>>>(b, x1, r, N, n1, c.hinv * c.hinv, e.Q, e.lam,
                                                                    omega, 0, tx, tx * tx);
  return hipGetLastError();
}

// ----------------------------------------------------------------- patch2d
// Q3 64^2 float32 11.5 -> 4.2 us (latency), 512^2 float32 22.1 -> 15.5,
// float64 33.3 -> 24.5, Q4 512^2 float64 120 -> 48 (a thread per patch or LDS
// passes over every patch's block before).
template <typename T, class S>
__global__ __launch_bounds__(S::NTH) void patch2d_kernel(const T* __restrict__ r, const T* __restrict__ xin,
                                                         T* __restrict__ xout, int N, int n1,
                                                         const T* __restrict__ Qg, const T* __restrict__ lamg,
                                                         T omega, int64_t zs, const int* __restrict__ active, int tx,
                                                         int total) {
  constexpr int K = S::K, TC = S::TC, NTH = S::NTH, BP = S::RS | 1;
  if (active && !active[blockIdx.z]) return;
  __shared__ T sA[cmax(S::RS * BP, S::SZU)];
  __shared__ T sM[S::SZM];
  __shared__ T sQ[4 * S::NN];
  __shared__ T sLam[4 * S::n];
  __shared__ T sD[S::NN];
  const int tile = tile2::xcd_order(blockIdx.x, total), bx = tile % tx, by = tile / tx;
  r += blockIdx.z * zs;
  xout += blockIdx.z * zs;
  if (xin) xin += blockIdx.z * zs;
  const int cx0 = bx * TC, cy0 = by * TC, NK = n1 - 1;
  tile2::Stage<T, T, S::RS, S::RS, BP, NTH> st;
  st.load(r, (cx0 - 1) * K + 1, (cy0 - 1) * K + 1, n1);
  tile2::StageEig<T, S::n, NTH> eig;
  eig.load(Qg, lamg);
  T xv[S::NO][K];
  const int rhi = min(cy0 * K + S::OWN, NK) - 1;
  const Rows<T> xi(xin ? xin : r, n1, cy0 * K, xin ? rhi : cy0 * K - 1);
#pragma unroll
  for (int q = 0; q < S::NO; ++q) {
    const int it = threadIdx.x + q * NTH, oy = it / TC, c = it - oy * TC;
    const bool on = it < S::OWN * TC && cx0 + c < N;
#pragma unroll
    for (int p = 0; p < K; ++p) xv[q][p] = xi.load(on ? xi.off(cy0 * K + oy, (cx0 + c) * K + p) : kOff);
  }
  st.store(sA);
  eig.store(sQ, sLam, sD);
  __syncthreads();
  const bool interior = cx0 >= 2 && cx0 + TC <= N - 2 && cy0 >= 2 && cy0 + TC <= N - 2;
  patch_phases<T, S>(sA, BP, sM, sA, Qg, sQ, sLam, sD, cx0, cy0, N, interior);
  zero_last<T, S::OWN, NTH>(xout, cx0 * K, cy0 * K, n1);
  const Rows<T> out(xout, n1, cy0 * K, rhi);
#pragma unroll
  for (int q = 0; q < S::NO; ++q) {
    const int it = threadIdx.x + q * NTH, oy = it / TC, c = it - oy * TC;
    if ((S::OWN * TC) % NTH != 0 && it >= S::OWN * TC) break;
    T a[K];
    corrections<T, S>(sA, a, Qg, sQ, oy, c, cx0, N, interior);
    write_owned<T, S>(out, xv[q], a, omega, oy, c, cx0, cy0, N);
  }
}

template <typename T, int K, int TC, int NTH>
hipError_t patch2d_g(int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega, hipStream_t s,
                     int nsys, int64_t zs, const int* active) {
  const int n1 = K * N + 1, tx = (N + TC - 1) / TC;
  patch2d_kernel<T, Fd<K, TC, NTH>><<<dim3(tx * tx, 1, nsys), NTH, 0, s>>>(r, xin, xout, N, n1, e.Q, e.lam, omega,
                                                                          zs, active, tx, tx * tx);
  return hipGetLastError();
}

// ------------------------------------------------------------------ dispatch
// Tiles (owned cells per side, threads) per degree and type, by sweeps over
// tile sizes and thread counts at 16^2 .. 512^2 cells.  Large: on meshes with
// at least one such tile per compute unit, where the redundant work of small
// tiles costs most.  Small: below that one workgroup's latency sets the time.
// k <= 4 takes large tiles (12 cells; 6 in Q3 float64, where LDS limits the
// workgroups per compute unit); from k = 5 on the LDS of one tile does.
// S(x, b) at 256^2 in us, large against small tile: float32 Q3 9.7 and 12.5,
// Q4 18.5 and 20.4, Q5 27 and 51, Q6 53 and 94, Q7 74 and 234; float64 Q3 15.6
// and 20.0, Q4 30 and 38, Q5 62 and 119, Q7 247 and 437, but Q6 184 and 171
// (the bases overflow the registers of the large tile).
template <int TC_, int NTH_, int CW_>
struct Tile {
  static constexpr int TC = TC_, NTH = NTH_, CW = CW_;
};
template <typename T, int K> struct StepTile;
template <typename T> struct StepTile<T, 2> { using Large = Tile<12, 512, 2>; using Small = Tile<4, 128, 1>; };
template <> struct StepTile<float, 3> { using Large = Tile<12, 512, 2>; using Small = Tile<4, 256, 1>; };
template <> struct StepTile<double, 3> { using Large = Tile<6, 256, 2>; using Small = Tile<4, 256, 1>; };
template <typename T> struct StepTile<T, 4> { using Large = Tile<12, 512, 2>; using Small = Tile<4, 256, 1>; };
template <typename T> struct StepTile<T, 5> { using Large = Tile<8, 512, 1>; using Small = Tile<4, 512, 1>; };
template <typename T> struct StepTile<T, 6> { using Large = Tile<6, 256, 1>; using Small = Tile<4, 512, 1>; };
template <> struct StepTile<float, 7> { using Large = Tile<8, 512, 1>; using Small = Tile<2, 256, 1>; };
template <> struct StepTile<double, 7> { using Large = Tile<4, 512, 1>; using Small = Tile<2, 256, 1>; };

template <typename T, int K> struct PatchTile;
template <typename T> struct PatchTile<T, 2> { using Large = Tile<15, 512, 1>; using Small = Tile<4, 128, 1>; };
template <typename T> struct PatchTile<T, 3> { using Large = Tile<8, 256, 1>; using Small = Tile<4, 256, 1>; };
template <typename T> struct PatchTile<T, 4> { using Large = Tile<8, 256, 1>; using Small = Tile<4, 256, 1>; };
template <typename T> struct PatchTile<T, 5> { using Large = Tile<6, 256, 1>; using Small = Tile<4, 320, 1>; };
template <typename T> struct PatchTile<T, 6> { using Large = Tile<6, 256, 1>; using Small = Tile<4, 320, 1>; };
template <> struct PatchTile<float, 7> { using Large = Tile<4, 128, 1>; using Small = Tile<2, 128, 1>; };
template <> struct PatchTile<double, 7> { using Large = Tile<2, 128, 1>; using Small = Tile<2, 128, 1>; };

template <typename T, int K> struct PreTile { using Small = Tile<4, 512, 1>; };
template <typename T> struct PreTile<T, 2> { using Small = Tile<8, 512, 1>; };
template <typename T> struct PreTile<T, 3> { using Small = Tile<6, 512, 1>; };
template <> struct PreTile<float, 4> { using Small = Tile<6, 512, 1>; };

inline bool fills(int N, int TC, int nsys) {
  const int64_t t = (N + TC - 1) / TC;
  return t * t * nsys >= 256;
}

// variant: 0 = by the mesh, 1 = the small tile, 2 = the large one (which c0ip_set_variant and the autotuner offer up to
// k = 3, where the tables' kernel has three tiles; for this kernel the autotuner times one of the two tiles twice).
template <typename T, int K>
hipError_t step2d_k(int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* x, const T* b, T* xout, T omega,
                    hipStream_t s, int nsys, int64_t zs, const int* active, int variant, const T* ec, int64_t zc) {
  using L = typename StepTile<T, K>::Large;
  using M = typename StepTile<T, K>::Small;
  if (variant == 2 || (variant != 1 && fills(N, L::TC, nsys)))
    return step2d_g<T, K, L::TC, L::NTH, L::CW>(N, c, e, x, b, xout, omega, s, nsys, zs, active, ec, zc);
  return step2d_g<T, K, M::TC, M::NTH, M::CW>(N, c, e, x, b, xout, omega, s, nsys, zs, active, ec, zc);
}

template <typename T, int K>
hipError_t pre2d_k(int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b, T* x1, T* r, T omega,
                   hipStream_t s) {
  if constexpr (K > 5) {
    return hipErrorNotSupported;
  } else {
    using M = typename PreTile<T, K>::Small;
    return pre2d_g<T, K, M::TC, M::NTH, M::CW>(N, c, e, b, x1, r, omega, s);
  }
}

template <typename T, int K>
hipError_t patch2d_k(int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega, hipStream_t s,
                     int nsys, int64_t zs, const int* active) {
  using L = typename PatchTile<T, K>::Large;
  using M = typename PatchTile<T, K>::Small;
  if (fills(N, L::TC, nsys)) return patch2d_g<T, K, L::TC, L::NTH>(N, e, r, xin, xout, omega, s, nsys, zs, active);
  return patch2d_g<T, K, M::TC, M::NTH>(N, e, r, xin, xout, omega, s, nsys, zs, active);
}

}  // namespace

template <typename T>
hipError_t launch_step2d(int k, int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* x, const T* b, T* xout,
                         T omega, hipStream_t s, int nsys, int64_t zs, const int* active, int variant, const T* ec,
                         int64_t zc) {
#define CALL(K) step2d_k<T, K>(N, c, e, x, b, xout, omega, s, nsys, zs, active, variant, ec, zc)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

template <typename T>
hipError_t launch_pre2d_ref(int k, int N, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b, T* x1, T* r, T omega,
                            hipStream_t s) {
#define CALL(K) pre2d_k<T, K>(N, c, e, b, x1, r, omega, s)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

template <typename T>
hipError_t launch_patch2d(int k, int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega,
                          hipStream_t s, int nsys, int64_t zs, const int* active) {
#define CALL(K) patch2d_k<T, K>(N, e, r, xin, xout, omega, s, nsys, zs, active)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

}  // namespace c0ip
