// One colour of the 2D coloured multiplicative smoother for the default
// penalty (Sec. 3, Fig. 2), in place:
//   x <- x + omega * sum_{v of the colour} R_v^T (local inverse) R_v (b - A x).
// The patches of a colour share no node and no entry of A couples two of
// them, so each is solved once and its correction added with a plain store.
//
// A group of TP lanes owns a patch from its first load to its last store.
// The (4k+1)^2 nodes of x around the vertex are staged in LDS (the residual on
// the patch's (2k-1)^2 interior nodes reaches no further), an x pass and a y
// pass with compile-time coefficients give the residual (lane = (row or
// column, one of the patch's two cells)), and the local solve takes one node
// per lane and transform.  Up to k = 4 a patch's lanes lie in one wave, so the
// phases need no workgroup barrier.  Why in place is safe: patches of one
// colour lie 4 cells apart along an axis or 2 along both, so the nodes that a
// patch's residual depends on (its closed rows and columns, extended by one
// cell) hold no interior node of another one; what is staged beyond them is
// not used.
#include "kernels.h"
#include "mvs2d.h"
#include "tile2d.h"

namespace c0ip {
namespace {

using ref::band_ref;
using tile::variant;

template <int K>
struct Grp {
  static constexpr int n = 2 * K - 1, NN = n * n, C = 2 * K + 1, W = 4 * K + 1;
  static constexpr int NEED = 2 * W > NN ? 2 * W : NN;  // lanes: x pass items, nodes
  static constexpr bool WAVE = NEED <= 64;
  static constexpr int PER = WAVE ? 64 / NEED : 1;                                   // patches per wave
  static constexpr int TP = WAVE ? 64 / PER : (NEED <= 85 ? 85 : NEED <= 128 ? 128 : 256);  // lanes per patch
  static constexpr int NTH = 256, NP = WAVE ? 4 * PER : NTH / TP;
  static constexpr int SZ = W * W + W * n + 2 * C * n + 2 * NN;  // LDS elements per patch
};

// Orders a patch's LDS writes before its following reads.
template <bool WAVE>
__device__ __forceinline__ void patch_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// 2D Q3 256^2 float64, 8 colours: 139 -> 73 us; the table kernel spent it on workgroup-wide
// phases whose every product waits for a coefficient from LDS.
template <typename T, int K, bool EXACT>
__global__ __launch_bounds__(Grp<K>::NTH) void mvs2d_colour_ref_kernel(
    const T* __restrict__ b, T* __restrict__ x, int N, int n1, ColourRows cr, int px, int py, T scale,
    const T* __restrict__ rsrc, const T* __restrict__ Qg, const T* __restrict__ lamg, const T* __restrict__ Aex,
    T omega) {
  using G = Grp<K>;
  constexpr int n = G::n, NN = G::NN, C = G::C, W = G::W, TP = G::TP, NTH = G::NTH;
  constexpr bool WAVE = G::WAVE;
  __shared__ T pool[G::NP * G::SZ];
  __shared__ T sQ[EXACT ? 1 : 4 * NN];
  __shared__ T sLam[EXACT ? 1 : 4 * n];
  // this thread's patch and its lane there
  const int t = threadIdx.x;
  const int slot = WAVE ? (t >> 6) * G::PER + (t & 63) / TP : t / TP;
  const int lane = WAVE ? (t & 63) % TP : t - slot * TP;
  const int q = blockIdx.x * G::NP + slot;
  const bool on = slot < G::NP && (!WAVE || (t & 63) < G::PER * TP) && q < cr.total;
  int vx = 1, vy = 1;
  if (on) colour_vertex(cr, px, py, q, vx, vy);
  const int sl = slot < G::NP ? slot : 0;
  T* sX = pool + sl * G::SZ;   // nodes (vy-2)K .. (vy+2)K, (vx-2)K .. (vx+2)K
  T* sTM = sX + W * W;         // X M_x on all rows, at the patch's interior columns
  T* sTL = sTM + W * n;        // X L_x and X B_x on the closed patch rows
  T* sTB = sTL + C * n;
  T* sA = sTB + C * n;
  T* sB = sA + NN;
  const int NK = n1 - 1;
  // loads first: eigendata, this lane's node of x (and of the given residual), b of its y items, the window of x
  constexpr int LQ = EXACT ? 1 : (4 * NN + NTH - 1) / NTH;
  T qv[LQ], lv = 0;
  if constexpr (!EXACT) {
#pragma unroll
    for (int u = 0; u < LQ; ++u) qv[u] = t + u * NTH < 4 * NN ? Qg[t + u * NTH] : T(0);
    if (t < 4 * n) lv = lamg[t];
  }
  const bool node = on && lane < NN;
  const int na = lane / n, nc = lane - na * n;
  const size_t gm = (size_t)((vy - 1) * K + 1 + na) * n1 + (vx - 1) * K + 1 + nc;
  const T xm = node ? x[gm] : T(0);
  const T rm = node && rsrc ? rsrc[gm] : T(0);
  const bool yit = on && lane < 2 * n;
  const int yc = lane >> 1, yh = lane & 1;  // column, cell
  constexpr int NS = (W * W + TP - 1) / TP;
  T bq[K], v[NS];
  if (!rsrc) {
#pragma unroll
    for (int p = 0; p < K; ++p)
      bq[p] = yit && (yh || p) ? b[(size_t)((vy - 1 + yh) * K + p) * n1 + (vx - 1) * K + 1 + yc] : T(0);
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int e = lane + u * TP, i = e / W, j = e - i * W;
      const int gy = (vy - 2) * K + i, gx = (vx - 2) * K + j;
      v[u] = on && lane < TP && e < W * W && gy >= 1 && gy < NK && gx >= 1 && gx < NK ? x[(size_t)gy * n1 + gx] : T(0);
    }
  }
  if constexpr (!EXACT) {
#pragma unroll
    for (int u = 0; u < LQ; ++u)
      if (t + u * NTH < 4 * NN) sQ[t + u * NTH] = qv[u];
    if (t < 4 * n) sLam[t] = lv;
  }
  if (rsrc) {
    if (node) sB[lane] = rm;
    __syncthreads();
  } else {
    if (on) {
#pragma unroll
      for (int u = 0; u < NS; ++u)
        if (lane + u * TP < W * W) sX[lane + u * TP] = v[u];
    }
    __syncthreads();  // (also the eigendata)
    // x pass: row i, cell h of the patch; the vertex column belongs to the second cell
    if (on && lane < 2 * W) {
      const int i = lane >> 1, h = lane & 1;
      T in[4 * K + 1];
#pragma unroll
      for (int j = 0; j <= 4 * K; ++j) {
        const int c = h * K + j - K;
        in[j] = sX[i * W + (c < 0 ? 0 : c)];  // c < 0: used by the first cell's p = 0 only, which is dropped
      }
      const T* w = in + 2 * K;
      T a[K];
      const int o = h ? K - 1 : -1;  // interior column of p = 0
#pragma unroll
      for (int p = 0; p < K; ++p) a[p] = band_ref<T, 0, K>(w + p, p);
#pragma unroll
      for (int p = 0; p < K; ++p)
        if (p > 0 || h) sTM[i * n + o + p] = a[p];
      if (i >= K && i <= 3 * K) {
#pragma unroll
        for (int p = 0; p < K; ++p) a[p] = band_ref<T, 1, K>(w + p, p);
#pragma unroll
        for (int p = 0; p < K; ++p)
          if (p > 0 || h) sTL[(i - K) * n + o + p] = a[p];
#pragma unroll
        for (int p = 0; p < K; ++p) a[p] = band_ref<T, 2, K>(w + p, p);
        ref::boundary_b<T, K>(a, w, vx - 1 + h, N);
#pragma unroll
        for (int p = 0; p < K; ++p)
          if (p > 0 || h) sTB[(i - K) * n + o + p] = a[p];
      }
    }
    patch_sync<WAVE>();
    // y pass: column yc, cell yh
    if (yit) {
      T acc[K], s[4 * K + 1], a[K];
#pragma unroll
      for (int j = 0; j <= 2 * K; ++j) {
        const int r = yh * K + j - K;
        s[j] = sTB[(r < 0 ? 0 : r) * n + yc];
      }
#pragma unroll
      for (int p = 0; p < K; ++p) acc[p] = band_ref<T, 0, K>(s + p + K, p);
#pragma unroll
      for (int j = 0; j <= 2 * K; ++j) {
        const int r = yh * K + j - K;
        s[j] = sTL[(r < 0 ? 0 : r) * n + yc];
      }
#pragma unroll
      for (int p = 0; p < K; ++p) acc[p] += T(2) * band_ref<T, 1, K>(s + p + K, p);
#pragma unroll
      for (int j = 0; j <= 4 * K; ++j) {
        const int r = yh * K + j - K;
        s[j] = sTM[(r < 0 ? 0 : r) * n + yc];
      }
#pragma unroll
      for (int p = 0; p < K; ++p) a[p] = band_ref<T, 2, K>(s + p + 2 * K, p);
      ref::boundary_b<T, K>(a, s + 2 * K, vy - 1 + yh, N);
#pragma unroll
      for (int p = 0; p < K; ++p)
        if (p > 0 || yh) sB[((yh ? K - 1 : -1) + p) * n + yc] = bq[p] - scale * (acc[p] + a[p]);
    }
    patch_sync<WAVE>();
  }
  T u = 0;
  if constexpr (EXACT) {
    // exact local solve: one dense row per lane
    if (node) {
      const T* row = Aex + (size_t)(variant(vy, N) * 4 + variant(vx, N)) * NN * NN + (size_t)lane * NN;
      for (int j = 0; j < NN; ++j) u += row[j] * sB[j];
    }
  } else {
    // r (sB) -> Q_x^T (sA) -> Q_y^T, reciprocal eigenvalue sums (sB) -> Q_y (sA) -> Q_x
    const int tx = variant(vx, N), ty = variant(vy, N);
    const T* qx = sQ + tx * NN;
    const T* qy = sQ + ty * NN;
    if (node) {
      T s = 0;
#pragma unroll
      for (int j = 0; j < n; ++j) s += qx[j * n + nc] * sB[na * n + j];
      sA[lane] = s;
    }
    patch_sync<WAVE>();
    if (node) {
      T s = 0;
#pragma unroll
      for (int j = 0; j < n; ++j) s += qy[j * n + na] * sA[j * n + nc];
      sB[lane] = s / (sLam[tx * n + nc] + sLam[ty * n + na]);
    }
    patch_sync<WAVE>();
    if (node) {
      T s = 0;
#pragma unroll
      for (int j = 0; j < n; ++j) s += qy[na * n + j] * sB[j * n + nc];
      sA[lane] = s;
    }
    patch_sync<WAVE>();
    if (node) {
#pragma unroll
      for (int j = 0; j < n; ++j) u += qx[nc * n + j] * sA[na * n + j];
    }
  }
  if (node) x[gm] = xm + omega * u;
}

template <typename T, int K, bool EXACT>
hipError_t mvs2d_ref_k(int N, int colour, const LevelCoef<T>& c, const T* Q, const T* lam, const T* Aex, const T* b,
                       const T* r, T* x, T omega, hipStream_t s) {
  const ColourRows cr = colour_rows(N, colour);
  if (cr.total <= 0) return hipSuccess;
  const int nblk = (cr.total + Grp<K>::NP - 1) / Grp<K>::NP;
  mvs2d_colour_ref_kernel<T, K, EXACT><<<nblk, Grp<K>::NTH, 0, s>>>(b, x, N, K * N + 1, cr, colour & 1,
                                                                   (colour >> 1) & 1, c.hinv * c.hinv, r, Q, lam,
                                                                   Aex, omega);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_mvs2d_colour_ref(int k, int N, int colour, const LevelCoef<T>& c, const T* Q, const T* lam,
                                   const T* Aex, const T* b, const T* r, T* x, T omega, hipStream_t s) {
#define CALL(K)                                                                     \
  (Aex ? mvs2d_ref_k<T, K, true>(N, colour, c, Q, lam, Aex, b, r, x, omega, s) \
       : mvs2d_ref_k<T, K, false>(N, colour, c, Q, lam, Aex, b, r, x, omega, s))
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

template hipError_t launch_mvs2d_colour_ref<double>(int, int, int, const LevelCoef<double>&, const double*,
                                                    const double*, const double*, const double*, const double*,
                                                    double*, double, hipStream_t);
template hipError_t launch_mvs2d_colour_ref<float>(int, int, int, const LevelCoef<float>&, const float*,
                                                   const float*, const float*, const float*, const float*, float*,
                                                   float, hipStream_t);

}  // namespace c0ip
