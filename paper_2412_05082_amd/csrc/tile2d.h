// Building blocks of the 2D tile kernels (default penalty): the operator on
// a tile of whole cells staged in LDS, and the fast-diagonalisation patch
// solves of a tile's patches.
//
// Operator: with X[j][i] (i = x index, fastest)
//   Y = M_y (X B_x) + 2 L_y (X L_x) + B_y (X M_x).
// One x pass per window of an input row writes X M_x, X L_x and X B_x to
// three LDS buffers, one y pass per column and cell combines them: two
// barriers and about 8 + 11 LDS accesses per node at k = 3.  Coefficients
// are the compile-time reference rows (refband.h) on every tile: no table in
// LDS or scalar loads to wait for, and no slower path for boundary tiles.
//
// Patch solves (eq. inverse): the sums over overlapping patches commute with
// the transforms along the other axis, so each row is transformed along x
// once per patch column (not once per patch), the y solves run in registers
// with one thread per (patch, x mode), and the transform back along x sums
// the (at most 2 x 2) patches of a node on the way out.  Three phases instead
// of three passes over every patch's block and a gather.
#pragma once

#include <hip/hip_runtime.h>

#include "rawbuf.h"
#include "refband.h"
#include "tiles.h"

namespace c0ip {
namespace tile2 {

using ref::band_ref;
using ref::mad;
using tile::Band;

// XCD-aware tile order: each XCD walks a contiguous band of the tiles.
__device__ __forceinline__ int xcd_order(int L, int total) {
  const int c = L & 7;
  return c * (total >> 3) + min(c, total & 7) + (L >> 3);
}

// q / d as a high product with magic(d) = 2^32 / d rounded up (d = 1: 0
// stands for 2^32): exact while q d < 2^32, which tile numbers of meshes that
// fit in memory keep by far.  A division by a kernel argument would take some
// 40 vector instructions of every wave.
__host__ __device__ inline unsigned magic(unsigned d) { return d == 1 ? 0u : 0xffffffffu / d + 1; }
__device__ __forceinline__ unsigned quotient(unsigned q, unsigned m) { return m ? __umulhi(q, m) : q; }

// Operator tile: TXC x TYC cells, NTH threads, x items of CW cells.
template <int K_, int TXC_, int TYC_, int NTH_, int CW_>
struct Op {
  static constexpr int K = K_, TXC = TXC_, TYC = TYC_, NTH = NTH_, CW = CW_;
  static constexpr int H = 2 * K, TX = TXC * K, TY = TYC * K, RX = TX + 2 * H, RY = TY + 2 * H;
  static constexpr int RXP = RX | 1, TXP = TX | 1;  // odd LDS strides: lanes down a column hit distinct banks
  static constexpr int RB = RY - 2 * K;             // rows of X L_x and X B_x: [K, RY - K)
  static constexpr int SZX = RY * RXP, SZM = RY * TXP, SZB = RB * TXP, SZT = SZM + 2 * SZB;
  static constexpr int NY = TX * TYC, NI = (NY + NTH - 1) / NTH;  // y items (column, cell)
  static_assert(TXC % CW == 0, "x items must divide the tile");
};

// Rows [rlo, rhi] of a vector with n1 entries per row as a raw buffer: a
// load outside them reads 0 and a store is dropped, which replaces the bounds
// tests (kOff: an offset outside every buffer).  Offsets are bytes from the
// start of row rlo; rows below it give offsets that wrap to huge values.
using rawbuf::kOff;
template <typename T>
struct Rows {
  __amdgpu_buffer_rsrc_t r;
  int rlo, n1;
  __device__ __forceinline__ Rows(const T* p, int n1_, int rlo_, int rhi) : rlo(rlo_), n1(n1_) {
    const int cnt = rhi - rlo_ + 1;
    r = rawbuf::make(p + (size_t)rlo_ * n1_, cnt > 0 ? cnt * n1_ * (int)sizeof(T) : 0);
  }
  __device__ __forceinline__ unsigned off(int row, int col) const {
    return (unsigned)(((row - rlo) * n1 + col) * (int)sizeof(T));
  }
  __device__ __forceinline__ T load(unsigned o) const { return rawbuf::load<T>(r, o); }
  __device__ __forceinline__ void store(unsigned o, T v) const { rawbuf::store<T>(r, o, v); }
};

// Stage a W x HT window (first node (gx0, gy0)) of x in LDS rows of stride
// WP, 0 on and outside the boundary.  A thread keeps its column and steps
// whole rows (one add per load; addresses and bounds tests per element took
// as many instructions as the operator's products).  Every load is issued
// before the first LDS store.
template <typename Tin, typename T, int W, int HT, int WP, int NTH>
struct Stage {
  static constexpr int RPI = NTH / W, NL = (HT + RPI - 1) / RPI;
  static_assert(RPI >= 1, "a row per step at least");
  T v[NL];
  int r0, c0;
  __device__ __forceinline__ void load(const Tin* __restrict__ x, int gx0, int gy0, int n1) {
    r0 = threadIdx.x / W;
    c0 = threadIdx.x - r0 * W;
    const Rows<Tin> buf(x, n1, max(gy0, 1), min(gy0 + HT - 1, n1 - 2));
    const int gx = gx0 + c0;
    const bool on = r0 < RPI && gx >= 1 && gx <= n1 - 2;
    const unsigned o = buf.off(gy0 + r0, gx), step = (unsigned)(RPI * n1 * (int)sizeof(Tin));
#pragma unroll
    for (int q = 0; q < NL; ++q) v[q] = (T)buf.load(on ? o + q * step : kOff);
  }
  __device__ __forceinline__ void store(T* __restrict__ s) const {
#pragma unroll
    for (int q = 0; q < NL; ++q)
      if (r0 < RPI && ((HT % RPI == 0) || q + 1 < NL || r0 + q * RPI < HT)) s[(r0 + q * RPI) * WP + c0] = v[q];
  }
};

// X on the operator tile with its 2k halo.
template <typename Tin, typename T, class G>
using StageX = Stage<Tin, T, G::RX, G::RY, G::RXP, G::NTH>;

// x pass: sT = X M_x (all staged rows), then X L_x and X B_x (rows [K, RY - K)).
// Items (row, CW cells), rows fastest across lanes; cx0 = the tile's first cell.
template <typename T, class G>
__device__ __forceinline__ void op_x(const T* __restrict__ sX, T* __restrict__ sT, int cx0, int N) {
  constexpr int K = G::K, CW = G::CW, H = G::H;
  constexpr int W = Band<2, K>::win_hi() + (CW - 1) * K + 1;  // input window (B's reaches the lowest offset, 0)
  T* sTL = sT + G::SZM;
  T* sTB = sTL + G::SZB;
  for (int it = threadIdx.x; it < G::RY * (G::TXC / CW); it += G::NTH) {
    const int g = it / G::RY, r = it - g * G::RY;
    T in[W];
#pragma unroll
    for (int j = 0; j < W; ++j) in[j] = sX[r * G::RXP + g * CW * K + j];
#pragma unroll
    for (int w = 0; w < CW; ++w)
#pragma unroll
      for (int p = 0; p < K; ++p)
        sT[r * G::TXP + (g * CW + w) * K + p] = band_ref<T, 0, K>(in + (w * K + p + H), p);
    if (r >= K && r < G::RY - K) {
#pragma unroll
      for (int w = 0; w < CW; ++w) {
        const T* v = in + (w * K + H);
        const int o = (r - K) * G::TXP + (g * CW + w) * K;
        T a[K];
#pragma unroll
        for (int p = 0; p < K; ++p) {
          sTL[o + p] = band_ref<T, 1, K>(v + p, p);
          a[p] = band_ref<T, 2, K>(v + p, p);
        }
        ref::boundary_b<T, K>(a, v, cx0 + g * CW + w, N);
#pragma unroll
        for (int p = 0; p < K; ++p) sTB[o + p] = a[p];
      }
    }
  }
}

// y pass of column l, cell cy (cell c of the mesh): acc = h^2 (A X) on its K nodes.
template <typename T, class G>
__device__ __forceinline__ void op_y(const T* __restrict__ sT, T (&acc)[G::K], int l, int cy, int c, int N) {
  constexpr int K = G::K, TXP = G::TXP;
  const T* sTL = sT + G::SZM;
  const T* sTB = sTL + G::SZB;
  {
    T t[3 * K];
#pragma unroll
    for (int j = 0; j < 3 * K; ++j) t[j] = sTB[(cy * K + j) * TXP + l];
#pragma unroll
    for (int p = 0; p < K; ++p) acc[p] = band_ref<T, 0, K>(t + p + K, p);
  }
  {
    T t[3 * K];
#pragma unroll
    for (int j = 0; j < 3 * K; ++j) t[j] = sTL[(cy * K + j) * TXP + l];
#pragma unroll
    for (int p = 0; p < K; ++p) acc[p] += T(2) * band_ref<T, 1, K>(t + p + K, p);
  }
  {
    T t[5 * K], a[K];
#pragma unroll
    for (int j = 0; j < 5 * K; ++j) t[j] = sT[(cy * K + j) * TXP + l];
#pragma unroll
    for (int p = 0; p < K; ++p) a[p] = band_ref<T, 2, K>(t + p + 2 * K, p);
    ref::boundary_b<T, K>(a, t + 2 * K, c, N);
#pragma unroll
    for (int p = 0; p < K; ++p) acc[p] += a[p];
  }
}

// Patch solves of the (TC+1)^2 patches touching a tile of TC x TC owned cells
// (n = 2k-1).  P patch columns; a row has XW = P n x modes.
template <int K_, int TC_, int NTH_>
struct Fd {
  static constexpr int K = K_, TC = TC_, NTH = NTH_, n = 2 * K - 1, NN = n * n, P = TC + 1;
  static constexpr int XW = P * n, XP = XW | 1, RS = (TC + 2) * K - 1, OWN = TC * K;
  static constexpr int SZM = RS * XP, SZU = P * n * XP;
  static constexpr int NO = (OWN * TC + NTH - 1) / NTH;  // output items (row, cell) per thread
};

// Eigenbases (4 variants), eigenvalues, and the interior patch's reciprocal
// eigenvalue sums sD[my][mx]; global loads first.
template <typename T, int n, int NTH>
struct StageEig {
  static constexpr int NN = n * n, LQ = (4 * NN + NTH - 1) / NTH, LL = (4 * n + NTH - 1) / NTH,
                       LD = (NN + NTH - 1) / NTH;
  T q[LQ], l[LL], da[LD], db[LD];
  __device__ __forceinline__ void load(const T* __restrict__ Qg, const T* __restrict__ lamg) {
#pragma unroll
    for (int u = 0; u < LQ; ++u) q[u] = (int)threadIdx.x + u * NTH < 4 * NN ? Qg[threadIdx.x + u * NTH] : T(0);
#pragma unroll
    for (int u = 0; u < LL; ++u) l[u] = (int)threadIdx.x + u * NTH < 4 * n ? lamg[threadIdx.x + u * NTH] : T(0);
#pragma unroll
    for (int u = 0; u < LD; ++u) {
      const int e = threadIdx.x + u * NTH;
      da[u] = e < NN ? lamg[e % n] : T(1);
      db[u] = e < NN ? lamg[e / n] : T(1);
    }
  }
  __device__ __forceinline__ void store(T* __restrict__ sQ, T* __restrict__ sLam, T* __restrict__ sD) const {
#pragma unroll
    for (int u = 0; u < LQ; ++u)
      if ((int)threadIdx.x + u * NTH < 4 * NN) sQ[threadIdx.x + u * NTH] = q[u];
#pragma unroll
    for (int u = 0; u < LL; ++u)
      if ((int)threadIdx.x + u * NTH < 4 * n) sLam[threadIdx.x + u * NTH] = l[u];
#pragma unroll
    for (int u = 0; u < LD; ++u)
      if ((int)threadIdx.x + u * NTH < NN) sD[threadIdx.x + u * NTH] = ref::recip_sum(da[u], db[u]);
  }
};

// Offset of a basis as a scalar.  The empty statement keeps the loads of a
// basis from being shared between two uses: all of it would not fit the
// registers of a large one.
__device__ __forceinline__ int scalar(int v) {
  v = __builtin_amdgcn_readfirstlane(v);
  asm volatile("" : "+s"(v));
  return v;
}

// A basis (n x n values at offset o) for one more use.  From 256 registers on
// (k = 7 in float64) it is loaded again for every transform, a row at a time:
// S(x, b) Q7 256^2 469 -> 244 us, 64^2 31 -> 18.  Smaller ones are faster when
// the compiler keeps what it can (Q6 256^2 float64 183 against 204, Q7 256^2
// float32 74 against 85).
template <typename T, int n>
constexpr bool kBigBasis = n * n * (int)sizeof(T) / 4 > 256;
template <typename T, int n, bool INT>
__device__ __forceinline__ const T* basis(const T* q, int o) {
  if constexpr (kBigBasis<T, n>) {
    if constexpr (INT)
      o = scalar(o);
    else
      asm volatile("" : "+v"(o));
  }
  return q + o;
}


// One 1D transform: out[c] = sum_a Q[a][c] in[a] (FWD) or out[a] = sum_c Q[a][c] in[c].
template <typename T, int n, bool FWD>
__device__ __forceinline__ void tr1(const T* __restrict__ q, const T (&in)[n], T (&out)[n]) {
  if constexpr (FWD && kBigBasis<T, n>) {  // row after row of Q, like the other direction
#pragma unroll
    for (int i = 0; i < n; ++i) out[i] = q[i] * in[0];
#pragma unroll
    for (int j = 1; j < n; ++j) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < n; ++i) out[i] = mad(q[j * n + i], in[j], out[i]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < n; ++i) {
      if (kBigBasis<T, n>) __builtin_amdgcn_sched_barrier(0);
      T s = (FWD ? q[i] : q[i * n]) * in[0];
#pragma unroll
      for (int j = 1; j < n; ++j) s = mad(FWD ? q[j * n + i] : q[i * n + j], in[j], s);
      out[i] = s;
    }
  }
}

// x transform of every row for every patch column; item (row, px), rows
// fastest.  sR: node (0, 0) of the patches' rows, row stride rp.  INT: every
// patch of the tile has the interior basis q0 (wave-uniform reads).
template <typename T, class S, bool INT>
__device__ __forceinline__ void fd_x(const T* __restrict__ sR, int rp, T* __restrict__ sM, const T* __restrict__ q0,
                                     const T* __restrict__ sQ, int cx0, int N) {
  constexpr int n = S::n;
  for (int it = threadIdx.x; it < S::P * S::RS; it += S::NTH) {
    const int px = it / S::RS, row = it - px * S::RS;
    T in[n], out[n];
#pragma unroll
    for (int a = 0; a < n; ++a) in[a] = sR[row * rp + px * S::K + a];
    tr1<T, n, true>(INT ? basis<T, n, true>(q0, 0) : basis<T, n, false>(sQ, tile::variant(cx0 + px, N) * S::NN), in, out);
#pragma unroll
    for (int a = 0; a < n; ++a) sM[row * S::XP + px * n + a] = out[a];
  }
}

// y solve of item (py, px, mx): transform along y, times the reciprocal
// eigenvalue sums, transform back; 0 for vertices outside the mesh.
template <typename T, class S, bool INT>
__device__ __forceinline__ void fd_y(const T* __restrict__ sM, T* __restrict__ sU, const T* __restrict__ q0,
                                     const T* __restrict__ sQ, const T* __restrict__ sLam,
                                     const T* __restrict__ sD, int cx0, int cy0, int N) {
  constexpr int n = S::n;
  for (int it = threadIdx.x; it < S::P * S::XW; it += S::NTH) {
    const int py = it / S::XW, col = it - py * S::XW, px = col / n, mx = col - px * n;
    const int vx = cx0 + px, vy = cy0 + py;
    T in[n], w[n];
    if (INT || (vx >= 1 && vx <= N - 1 && vy >= 1 && vy <= N - 1)) {
      const int ty = INT ? 0 : tile::variant(vy, N);
      const T lx = sLam[(INT ? 0 : tile::variant(vx, N)) * n + mx];
      const T* q = INT ? basis<T, n, true>(q0, 0) : basis<T, n, false>(sQ, ty * S::NN);
#pragma unroll
      for (int a = 0; a < n; ++a) in[a] = sM[(py * S::K + a) * S::XP + col];
      tr1<T, n, true>(q, in, w);
#pragma unroll
      for (int m = 0; m < n; ++m) w[m] *= INT ? sD[m * n + mx] : ref::recip_sum(lx, sLam[ty * n + m]);
      if (kBigBasis<T, n>) q = INT ? basis<T, n, true>(q0, 0) : basis<T, n, false>(sQ, ty * S::NN);
      tr1<T, n, false>(q, w, in);
    } else {
#pragma unroll
      for (int a = 0; a < n; ++a) in[a] = T(0);
    }
#pragma unroll
    for (int a = 0; a < n; ++a) sU[(py * n + a) * S::XP + col] = in[a];
  }
}

// Corrections of the K nodes of owned row oy, cell c: the patches containing
// them are summed along y, transformed back along x and summed along x.
template <typename T, class S, bool INT>
__device__ __forceinline__ void fd_out(const T* __restrict__ sU, T (&out)[S::K], const T* __restrict__ q0,
                                       const T* __restrict__ sQ, int oy, int c, int cx0, int N) {
  constexpr int K = S::K, n = S::n;
  const int my = oy / K, ry = oy - my * K;
  const T* ua = sU + (my * n + K - 1 + ry) * S::XP + c * n;
  const T* ub = sU + ((my + 1) * n + ry - 1) * S::XP + c * n;
  T wa[n], wb[n];
#pragma unroll
  for (int m = 0; m < n; ++m) {
    wa[m] = ua[m];
    wb[m] = ua[n + m];
  }
  if (ry > 0) {
#pragma unroll
    for (int m = 0; m < n; ++m) {
      wa[m] += ub[m];
      wb[m] += ub[n + m];
    }
  }
  const T* qa = INT ? basis<T, n, true>(q0, 0) : basis<T, n, false>(sQ, tile::variant(cx0 + c, N) * S::NN);
  const T* qb = INT ? basis<T, n, true>(q0, 0) : basis<T, n, false>(sQ, tile::variant(cx0 + c + 1, N) * S::NN);
#pragma unroll
  for (int p = 0; p < K; ++p) {
    if (kBigBasis<T, n>) __builtin_amdgcn_sched_barrier(0);
    T a = qa[(K - 1 + p) * n] * wa[0];
#pragma unroll
    for (int m = 1; m < n; ++m) a = mad(qa[(K - 1 + p) * n + m], wa[m], a);
    if (p > 0) {  // a sum of its own: one chain over both patches would round at the size of their sum
      T b = qb[(p > 0 ? p - 1 : 0) * n] * wb[0];
#pragma unroll
      for (int m = 1; m < n; ++m) b = mad(qb[(p > 0 ? p - 1 : 0) * n + m], wb[m], b);
      a += b;
    }
    out[p] = a;
  }
}

// sX += (P ec) on the operator tile's staged region, for tiles whose first
// cell is even + 1 (the fused smoother's): the coarse cells covering it are
// staged in sC, interpolated along x into sP, then along y.  Items are whole
// coarse cells, so the embedding table is compile-time.
template <typename T, class G>
struct Prolong {
  static constexpr int K = G::K, NC = (G::TXC + 6) / 2, CX = NC * K + 1, CP = CX | 1, NTH = G::NTH;
  static constexpr int SZC = CX * CP, SZP = CX * G::RXP;
  static_assert(G::TXC == G::TYC && G::TXC % 2 == 0, "the fused smoother's tiles");
  Stage<T, T, CX, CX, CP, NTH> st;
  __device__ __forceinline__ void load(const T* __restrict__ ec, int cxt, int cyt, int N) {
    // first staged fine cell cxt - 2 (odd): coarse cells from (cxt - 3) / 2
    st.load(ec, (cxt - 3) / 2 * K, (cyt - 3) / 2 * K, K * (N / 2) + 1);
  }
  __device__ __forceinline__ void store(T* __restrict__ sC) const { st.store(sC); }
  static __device__ __forceinline__ void along_x(const T* __restrict__ sC, T* __restrict__ sP) {
    for (int it = threadIdx.x; it < CX * NC; it += NTH) {
      const int c = it / CX, r = it - c * CX;
      T in[K + 1];
#pragma unroll
      for (int a = 0; a <= K; ++a) in[a] = sC[r * CP + c * K + a];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int f = 2 * c + s - 1;  // fine cell within the staged region
        if (f < 0 || f >= G::TXC + 4) continue;
#pragma unroll
        for (int p = 0; p < K; ++p) {
          T v = (T)RefCoef<K>::pt[s][p][0] * in[0];
#pragma unroll
          for (int a = 1; a <= K; ++a) v = mad((T)RefCoef<K>::pt[s][p][a], in[a], v);
          sP[r * G::RXP + f * K + p] = v;
        }
      }
    }
  }
  static __device__ __forceinline__ void along_y(const T* __restrict__ sP, T* __restrict__ sX) {
    for (int it = threadIdx.x; it < G::RX * NC; it += NTH) {
      const int c = it / G::RX, col = it - c * G::RX;
      T in[K + 1];
#pragma unroll
      for (int a = 0; a <= K; ++a) in[a] = sP[(c * K + a) * G::RXP + col];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int f = 2 * c + s - 1;
        if (f < 0 || f >= G::TYC + 4) continue;
#pragma unroll
        for (int p = 0; p < K; ++p) {
          T v = (T)RefCoef<K>::pt[s][p][0] * in[0];
#pragma unroll
          for (int a = 1; a <= K; ++a) v = mad((T)RefCoef<K>::pt[s][p][a], in[a], v);
          sX[(f * K + p) * G::RXP + col] += v;
        }
      }
    }
  }
};

// Transfers, with the compile-time embedding table pt[s][p][a] (value of coarse
// basis a at the fine node of position p in fine cell s of the coarse cell).
// The k coarse values of a cell from the fine nodes of its left neighbour and its own (in[0..4k-1]).
template <typename T, int K>
__device__ __forceinline__ void gather(const T* in, T (&o)[K]) {
#pragma unroll
  for (int a = 0; a < K; ++a) {
    T v = 0;
#pragma unroll
    for (int q = 0; q < 2 * K; ++q) v = mad((T)RefCoef<K>::pt[q / K][q % K][a], in[2 * K + q], v);
    if (a == 0) {
#pragma unroll
      for (int q = 0; q < 2 * K; ++q) v = mad((T)RefCoef<K>::pt[q / K][q % K][K], in[q], v);
    }
    o[a] = v;
  }
}

// The 2k fine values of a coarse cell from its k + 1 nodes.
template <typename T, int K>
__device__ __forceinline__ void spread(const T* in, T (&o)[2 * K]) {
#pragma unroll
  for (int q = 0; q < 2 * K; ++q) {
    T v = 0;
#pragma unroll
    for (int a = 0; a <= K; ++a) v = mad((T)RefCoef<K>::pt[q / K][q % K][a], in[a], v);
    o[q] = v;
  }
}

}  // namespace tile2
}  // namespace c0ip
