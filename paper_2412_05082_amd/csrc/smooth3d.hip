// 3D additive vertex-patch smoother for gfx950, streaming along z (Sec. 3,
// the AVS definition with eq. localsolverbila in 3D, inverted by fast
// diagonalisation, eq. inverse):
//   x_out = x_in + omega sum_v R_v^T (Q (x) Q (x) Q) (L_x + L_y + L_z)^-1
//                                    (Q (x) Q (x) Q)^T R_v r.
// A workgroup owns a TC x TC tile of cells in x, y (owner computes) over a
// chunk of z cells, and walks the vertex layers vz of the chunk.  The
// patches of a layer are the (TC+1)^2 patches around the tile's vertices;
// each covers 2k-1 residual planes, of which k-1 are shared with the next
// layer.  The sums over overlapping patches commute with the inverse
// transforms of the other axes, so every 1D transform runs once per plane
// and not once per (layer, plane):
//   * k new residual planes are staged in LDS (the next k are already in
//     flight in registers);
//   * x: every (plane, row, patch column px) is transformed once, for the
//     patches of all rows py that share it, into LDS;
//   * y and z: thread (px, py, mx) owns the x mode mx of one patch column.
//     It transforms along y in registers, keeps the 2k-1 planes of its
//     n = 2k-1 y modes in a register window, and per layer transforms along
//     z, scales by the tabulated reciprocal eigenvalue sums, transforms back
//     and adds to a second window, the sum over the layers of the output
//     planes.  The k lowest planes are then complete; they are transformed
//     back along y into LDS;
//   * each (plane, row, cell) item sums the (at most 2 x 2) patches that
//     contain its row and cell, transforms back along x and writes its k
//     nodes.
// Nothing but the staged planes and the x-y modes passes through LDS: about
// 20 accesses per DoF for k = 3 (keeping every patch's block of a layer in
// LDS and running six passes over it took about 80).  All sums run in a
// fixed order (deterministic).
#include <algorithm>

#include "faces3d.h"
#include "kernels.h"
#include "rawbuf.h"
#include "refband.h"

namespace c0ip {
namespace {

// variant of the patch at vertex v in [1, N-1] along one axis (0 interior,
// 1 touching the lower boundary, 2 the upper one, 3 both)
__device__ __forceinline__ int pvariant(int v, int N) { return (v == 1 ? 1 : 0) | (v == N - 1 ? 2 : 0); }

template <int K_, int TC_>
struct SGeo {
  static constexpr int K = K_, TC = TC_, NTH = 256;
  static constexpr int n = 2 * K - 1, NN = n * n, P = TC + 1;
  static constexpr int RS = (TC + 2) * K - 1, RSP = RS | 1;  // staged residual plane: RS x RS nodes
  static constexpr int XW = P * n, XP = XW | 1;              // x modes of a row, odd LDS stride
  static constexpr int OWN = TC * K;                         // owned nodes per direction
  static constexpr int SZR = K * RS * RSP, SZX = K * RS * XP, SZU = K * P * n * XP;
  static_assert(P * P * n <= NTH, "one thread per x mode of a patch column");
};

// One 1D transform of n values: out[c] = sum_a Q[a][c] in[a] (FWD, Q^T) or
// out[a] = sum_c Q[a][c] in[c] (inverse).  Q is either wave-uniform (held in
// registers) or a per-lane row in LDS.
template <typename T, int n, bool FWD>
__device__ __forceinline__ void tr1(const T* q, const T (&in)[n], T (&out)[n]) {
#pragma unroll
  for (int i = 0; i < n; ++i) {
    T s = 0;
#pragma unroll
    for (int j = 0; j < n; ++j) s += (FWD ? q[j * n + i] : q[i * n + j]) * in[j];
    out[i] = s;
  }
}

template <typename T, class G, bool UNI>
__device__ __forceinline__ void smooth3d_tile(const T* __restrict__ r, const T* __restrict__ xin, T* __restrict__ xout,
                                              int N, const T* __restrict__ Qg, T omega, int cx0, int cy0, int c0,
                                              int c1, T* __restrict__ sR, T* __restrict__ sX, T* __restrict__ sU,
                                              const T* __restrict__ sQ, const T* __restrict__ sLam) {
  constexpr int K = G::K, TC = G::TC, n = G::n, NN = G::NN, P = G::P, NTH = G::NTH, RS = G::RS, RSP = G::RSP,
                XP = G::XP, OWN = G::OWN;
  const int n1 = K * N + 1, NK = n1 - 1;
  const size_t plane = (size_t)n1 * n1;
  const unsigned pbytes = (unsigned)(plane * sizeof(T));
  const int tid = threadIdx.x;
  // interior-variant eigenbasis in registers (wave-uniform)
  T q0[NN];
#pragma unroll
  for (int i = 0; i < NN; ++i) q0[i] = Qg[i];
  // staged residual plane: node offsets (kOff outside [1, NK-1]^2)
  constexpr int NR = (RS * RS + NTH - 1) / NTH;
  unsigned roff[NR];
#pragma unroll
  for (int t = 0; t < NR; ++t) {
    const int e = tid + t * NTH;
    const int j = e / RS, i = e - j * RS;
    const int gx = (cx0 - 1) * K + 1 + i, gy = (cy0 - 1) * K + 1 + j;
    roff[t] = (e < RS * RS && gx >= 1 && gx <= NK - 1 && gy >= 1 && gy <= NK - 1)
                  ? (unsigned)(gy * n1 + gx) * sizeof(T)
                  : rawbuf::kOff;
  }
  // this thread's x mode mx of patch column (px, py)
  const int py = tid / G::XW, col = tid - py * G::XW, px = col / n, mx = col - px * n;
  const int vx = cx0 + px, vy = cy0 + py;
  const bool mine = tid < P * G::XW;
  const bool valid = mine && vx >= 1 && vx <= N - 1 && vy >= 1 && vy <= N - 1;
  const T* qy = UNI ? q0 : sQ + (mine ? pvariant(vy, N) : 0) * NN;
  T win[n][n], acc[n][n], rec[n][n];  // [plane][y mode]; reciprocal sums [y mode][z mode]
#pragma unroll
  for (int j = 0; j < n; ++j)
#pragma unroll
    for (int m = 0; m < n; ++m) win[j][m] = acc[j][m] = rec[j][m] = T(0);
  int zrec = -1;  // z variant of rec
  const int v0 = max(c0, 1), vend = c1 == N ? N : c1;
  T v[K][NR];
  auto load = [&](int vz) {  // residual planes vz k .. vz k + k - 1 (0 beyond the interior)
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const int zp = vz * K + j;
      const __amdgpu_buffer_rsrc_t rr = rawbuf::make(r + (size_t)zp * plane, zp >= 1 && zp <= NK - 1 ? pbytes : 0u);
#pragma unroll
      for (int t = 0; t < NR; ++t) v[j][t] = rawbuf::load<T>(rr, roff[t]);
    }
  };
  load(v0 - 1);
  for (int vz = v0 - 1; vz <= vend; ++vz) {
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
      for (int t = 0; t < NR; ++t) {
        const int e = tid + t * NTH, row = e / RS;
        if (NR * NTH == RS * RS || e < RS * RS) sR[j * RS * RSP + e + row * (RSP - RS)] = v[j][t];
      }
    if (vz < vend) load(vz + 1);
    __syncthreads();
    // x transform of every row of the new planes (rows fastest across lanes)
    for (int it = tid; it < K * P * RS; it += NTH) {
      const int jp = it / RS, row = it - jp * RS, j = jp / P, qx = jp - j * P;
      const T* src = sR + (j * RS + row) * RSP + qx * K;
      T* dst = sX + (j * RS + row) * XP + qx * n;
      T in[n], out[n];
#pragma unroll
      for (int a = 0; a < n; ++a) in[a] = src[a];
      if (UNI)
        tr1<T, n, true>(q0, in, out);
      else
        tr1<T, n, true>(sQ + pvariant(cx0 + qx, N) * NN, in, out);
#pragma unroll
      for (int a = 0; a < n; ++a) dst[a] = out[a];
    }
    __syncthreads();
    // the window moves up by k planes; the new ones are transformed along y
#pragma unroll
    for (int j = 0; j < n; ++j)
#pragma unroll
      for (int m = 0; m < n; ++m) {
        if (j < K - 1) win[j][m] = win[j + K][m];
        acc[j][m] = j < K - 1 ? acc[j + K][m] : T(0);
      }
    if (valid) {
#pragma unroll
      for (int j = 0; j < K; ++j) {
        T in[n];
#pragma unroll
        for (int a = 0; a < n; ++a) in[a] = sX[(j * RS + py * K + a) * XP + col];
        tr1<T, n, true>(qy, in, win[K - 1 + j]);
      }
    }
    if (vz >= v0 && vz <= N - 1) {
      const int zv = pvariant(vz, N);
      const T* qz = Qg + zv * NN;
      if (zv != zrec) {
        zrec = zv;
        if (valid) {
          const T lx = sLam[pvariant(vx, N) * n + mx];
#pragma unroll
          for (int m = 0; m < n; ++m) {
            const T ly = sLam[pvariant(vy, N) * n + m], lxy = lx + ly, exy = ref::sum_error(lx, ly, lxy);
#pragma unroll
            for (int c = 0; c < n; ++c) {
              const T lz = sLam[zv * n + c], d = lxy + lz;
              rec[m][c] = ref::recip(d, exy + ref::sum_error(lxy, lz, d));
            }
          }
        }
      }
      if (valid) {
#pragma unroll
        for (int m = 0; m < n; ++m) {
          T in[n], w[n];
#pragma unroll
          for (int j = 0; j < n; ++j) in[j] = win[j][m];
          tr1<T, n, true>(qz, in, w);
#pragma unroll
          for (int c = 0; c < n; ++c) w[c] *= rec[m][c];
          tr1<T, n, false>(qz, w, in);
#pragma unroll
          for (int j = 0; j < n; ++j) acc[j][m] += in[j];
        }
      }
    }
    // planes (vz - 1) k + 1 .. vz k are complete (plane 0 is boundary)
    if (vz < v0 && c0 > 0) continue;
    if (mine) {
#pragma unroll
      for (int j = 0; j < K; ++j) {
        T u[n];
        tr1<T, n, false>(qy, acc[j], u);
#pragma unroll
        for (int a = 0; a < n; ++a) sU[((j * P + py) * n + a) * XP + col] = u[a];
      }
    }
    __syncthreads();
    for (int it = tid; it < K * OWN * TC; it += NTH) {
      const int jr = it / TC, c = it - jr * TC, j = jr / OWN, oy = jr - j * OWN;
      const int zp = (vz - 1) * K + 1 + j;
      const int gx = (cx0 + c) * K, gy = cy0 * K + oy;
      if (zp < c0 * K || zp >= c1 * K || gx >= NK || gy >= NK) continue;
      const size_t o = (size_t)zp * plane + (size_t)gy * n1 + gx;
      T xv[K];
#pragma unroll
      for (int p = 0; p < K; ++p) xv[p] = xin ? xin[o + p] : T(0);
      // patch row my (and my + 1 unless the node is on the vertex line)
      const int my = oy / K, ry = oy - my * K;
      const T* ua = sU + ((j * P + my) * n + K - 1 + ry) * XP + c * n;
      const T* ub = sU + ((j * P + my + 1) * n + ry - 1) * XP + c * n;
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
      const T* qa = UNI ? q0 : sQ + pvariant(cx0 + c, N) * NN;
      const T* qb = UNI ? q0 : sQ + pvariant(cx0 + c + 1, N) * NN;
#pragma unroll
      for (int p = 0; p < K; ++p) {
        T a = 0;
#pragma unroll
        for (int m = 0; m < n; ++m) a += qa[(K - 1 + p) * n + m] * wa[m];
        if (p > 0) {  // a sum of its own: one chain over both patches would round at the size of their sum
          T b = 0;
#pragma unroll
          for (int m = 0; m < n; ++m) b += qb[(p > 0 ? p - 1 : 0) * n + m] * wb[m];
          a += b;
        }
        const bool bnd = zp == 0 || gy == 0 || gx + p == 0;
        xout[o + p] = bnd ? T(0) : xv[p] + omega * a;
      }
    }
  }
}

// One workgroup per (tile, z chunk), each XCD walking a contiguous band of
// them (neighbouring tiles share halos in that XCD's L2), then the
// workgroups that zero the faces.  Bound by vector instructions (Q3 float32:
// they take 74 % of the SIMDs' issue slots).  3D Q3 128^3, this kernel alone:
// float32 891 -> 400 us with the register windows in place of six passes over
// every patch's block in LDS, float64 1826 -> 780 us.  The register bound
// holds Q3 float32 at 4 waves per SIMD (136 registers and 3 waves without it:
// S(x, b) 128^3 692 us against 630).  The other degrees and types are left to
// the compiler: Q2 stays at 4 waves and more, Q3 float64 and Q4 take 237 to all
// 256 registers, and a tighter bound would spill their windows.
template <typename T, class G>
__global__ __launch_bounds__(G::NTH, G::K == 3 && sizeof(T) == 4 ? 4 : 1) void smooth3d_kernel(const T* __restrict__ r, const T* __restrict__ xin,
                                                          T* __restrict__ xout, int N, const T* __restrict__ Qg,
                                                          const T* __restrict__ lamg, T omega, int tx, int nz,
                                                          int zcc) {
  const int n1 = G::K * N + 1;
  const int total = tx * tx * nz, L = blockIdx.x;
  if (L >= total) {
    zero_faces<T, G::NTH>(xout, n1, L - total);
    return;
  }
  __shared__ T sR[G::SZR];
  __shared__ T sX[G::SZX];
  __shared__ T sU[G::SZU];
  __shared__ T sQ[4 * G::NN];
  __shared__ T sLam[4 * G::n];
  for (int e = threadIdx.x; e < 4 * G::NN; e += G::NTH) sQ[e] = Qg[e];
  for (int e = threadIdx.x; e < 4 * G::n; e += G::NTH) sLam[e] = lamg[e];
  // (the first barrier of the layer loop orders these copies)
  const int xcd = L & 7, logical = xcd * (total >> 3) + min(xcd, total & 7) + (L >> 3);
  const int bx = logical % tx, rest = logical / tx, by = rest % tx, bz = rest / tx;
  const int cx0 = bx * G::TC, cy0 = by * G::TC;
  const int c0 = bz * zcc, c1 = min(c0 + zcc, N);
  // tiles whose patches are all interior in x and y take the basis in
  // scalar registers (when it fits them)
  constexpr bool kUniFits = G::NN * (int)sizeof(T) / 4 <= 50;
  const bool uni = kUniFits && cx0 >= 2 && cx0 + G::TC <= N - 2 && cy0 >= 2 && cy0 + G::TC <= N - 2;
  if constexpr (kUniFits) {
    if (uni) {
      smooth3d_tile<T, G, true>(r, xin, xout, N, Qg, omega, cx0, cy0, c0, c1, sR, sX, sU, sQ, sLam);
      return;
    }
  }
  smooth3d_tile<T, G, false>(r, xin, xout, N, Qg, omega, cx0, cy0, c0, c1, sR, sX, sU, sQ, sLam);
}

template <typename T, int K> struct SmoothCfg;
template <typename T> struct SmoothCfg<T, 2> { using G = SGeo<2, 8>; };
template <typename T> struct SmoothCfg<T, 3> { using G = SGeo<3, 6>; };
template <typename T> struct SmoothCfg<T, 4> { using G = SGeo<4, 5>; };

template <typename T, class G>
hipError_t smooth3d_g(int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega, hipStream_t s) {
  const int n1 = G::K * N + 1;
  const int tx = (N + G::TC - 1) / G::TC;
  // z chunks: about as many workgroups as the chip holds at once by the
  // kernel's registers and LDS (float32: 8, 4 and 2 per compute unit for
  // k = 2, 3, 4; float64 half of that): fewer leave it idle, more recompute
  // the patches shared between chunks (Q3 64^3 float32: 129 us with 512, 121
  // with 1024, 134 with 2048).  For k = 4 twice as many (Q4 64^3 float64: 990
  // us with 256, 856 with 512, 903 with 1024).  Small meshes go down to one
  // cell per chunk: there the march along z sets the time (Q4 16^3 float64,
  // which boxes take now: 54 us at 4 cells, 28 at 1).
  const int target = (G::K == 2 ? 2048 : 1024) / (sizeof(T) == 4 ? 1 : 2);
  int zcc = N;
  while (zcc > 1 && (int64_t)tx * tx * ((N + zcc - 1) / zcc) < target) zcc = (zcc + 1) / 2;
  const int nz = (N + zcc - 1) / zcc;
  smooth3d_kernel<T, G><<<tx * tx * nz + face_blocks<G::NTH>(n1), G::NTH, 0, s>>>(r, xin, xout, N, e.Q, e.lam, omega, tx, nz, zcc);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_patch3d(int k, int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega,
                          hipStream_t s) {
  // raw buffer offsets of a plane must stay below 2^31 bytes
  if ((double)(k * N + 1) * (k * N + 1) * sizeof(T) >= 2147483648.0) return hipErrorInvalidValue;
  switch (k) {
    case 2: return smooth3d_g<T, typename SmoothCfg<T, 2>::G>(N, e, r, xin, xout, omega, s);
    case 3: return smooth3d_g<T, typename SmoothCfg<T, 3>::G>(N, e, r, xin, xout, omega, s);
    case 4:
      // On small meshes the march along z, layer after layer in a few workgroups, sets the time: boxes
      // (smooth3d_box.hip). S(0, b) in us, march against boxes: float64 2^3 21.4 and 5.8, 8^3 27.1 and 11.6, 16^3 28.0
      // and 17.7, 32^3 132 and 99, 64^3 500 and 739; float32 2^3 15.8 and 5.8, 16^3 20.0 and 13.9, 32^3 71 and 69,
      // 64^3 220 and 496.
      if (N <= 32) return launch_patch3d_box<T>(k, N, e, r, xin, xout, omega, s);
      return smooth3d_g<T, typename SmoothCfg<T, 4>::G>(N, e, r, xin, xout, omega, s);
    default: return launch_patch3d_box<T>(k, N, e, r, xin, xout, omega, s);
  }
}

template hipError_t launch_patch3d<double>(int, int, const LevelEig<double>&, const double*, const double*,
                                           double*, double, hipStream_t);
template hipError_t launch_patch3d<float>(int, int, const LevelEig<float>&, const float*, const float*, float*,
                                          float, hipStream_t);

}  // namespace c0ip
