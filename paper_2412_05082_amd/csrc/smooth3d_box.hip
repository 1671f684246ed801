// 3D additive vertex-patch solves x_out = x_in + omega sum_v R_v^T A~_v^{-1} R_v r
// for k >= 5, and for k = 4 on small meshes, on boxes of cells (smooth3d.hip
// holds a patch's lines in registers along a march, which only fits up to
// k = 4, and whose layers follow one another).
//
// A workgroup owns TC x TC cells of one layer and solves the patches that
// touch them.  Sums over patches that overlap along one axis commute with the
// transforms along the others, so per z vertex of the layer (two) every column,
// row and line of the box is transformed once for all of its patches, in one
// LDS buffer that each phase rewrites in place, an item owning the line that
// it reads:
//   z: column of r -> n z modes              [z mode][y][x]
//   x: row -> n modes of each x vertex       [z mode][y][x mode]
//   y: line -> per y vertex n modes, reciprocal eigenvalue sums, back to the
//      owned y nodes                         [z mode][owned y][x mode]
//   x: row -> owned x nodes                  [z mode][owned y][owned x]
//   z: column -> owned nodes of the layer, added up over the z vertices in
//      registers.
// The bases are the same for a whole workgroup (they depend on the vertex along
// the axis alone): they come through scalar loads, a row at a time, and a
// product costs no LDS access.
//
// Solving patch by patch for every cell (8 patches each, bases in LDS) took,
// with the residual, 1124 us for a step at Q5 16^3 float64 against 67 now (39
// of them here), 17652 against 1824 at Q7 32^3.  Bound by the products'
// issue: about 780 per node at k = 5, 1100 at k = 7, where a box's LDS leaves
// one workgroup on a CU in float64.
#include "faces3d.h"
#include "kernels.h"
#include "tile2d.h"

namespace c0ip {
namespace {

using tile2::scalar;
using tile::variant;

template <int K> struct PatchBoxThreads;  // a y line per thread, whole waves
template <> struct PatchBoxThreads<4> { static constexpr int NTH = 192; };
template <> struct PatchBoxThreads<5> { static constexpr int NTH = 256; };
template <> struct PatchBoxThreads<6> { static constexpr int NTH = 384; };
template <> struct PatchBoxThreads<7> { static constexpr int NTH = 512; };

template <int K_>
struct PatchBox {
  static constexpr int K = K_, TC = 2, NTH = PatchBoxThreads<K>::NTH, n = 2 * K - 1;
  static constexpr int V = TC + 1, S = (TC + 2) * K - 1, M = V * n, TX = TC * K;  // vertices, nodes, modes, owned nodes
  static constexpr int MP = M | 1;                                                // odd LDS row stride
  static_assert(TX * TX <= NTH && S <= M, "an owned column per thread; rows hold nodes and modes");
};

template <typename T, int K, int NTH>
__global__ __launch_bounds__(NTH) void patch3d_box_kernel(const T* __restrict__ r, const T* xin, T* xout, int N,
                                                          int n1, const T* __restrict__ Qg,
                                                          const T* __restrict__ lamg, T omega, int nt, unsigned mt,
                                                          int total) {
  using G = PatchBox<K>;
  constexpr int TC = G::TC, n = G::n, NN = n * n, V = G::V, S = G::S, M = G::M, MP = G::MP, TX = G::TX;
  if ((int)blockIdx.x >= total) {
    zero_faces<T, NTH>(xout, n1, blockIdx.x - total);
    return;
  }
  __shared__ T pool[n * S * MP];
  __shared__ T sLam[4 * n];
  const unsigned q = tile2::xcd_order(blockIdx.x, total), yz = tile2::quotient(q, mt), cz_ = tile2::quotient(yz, mt);
  const int cx0 = (int)(q - yz * nt) * TC, cy0 = (int)(yz - cz_ * nt) * TC, cz = (int)cz_;
  const int t = threadIdx.x;
  const size_t pl = (size_t)n1 * n1;
  if (t < 4 * n) sLam[t] = lamg[t];
  T acc[K];
#pragma unroll
  for (int p = 0; p < K; ++p) acc[p] = T(0);
  for (int h = 0; h < 2; ++h) {
    const int vz = cz + h;
    if (vz < 1 || vz > N - 1) continue;  // the same for the whole workgroup
    const int tz = variant(vz, N);
    {
      // z forward
      const int ps = n1 * n1 * (int)sizeof(T), z0 = (vz - 1) * K + 1;
      const __amdgpu_buffer_rsrc_t buf =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(r) + z0 * pl, (short)0, n * ps, 0x00020000);
      for (int it = t; it < S * S; it += NTH) {
        const int j = it / S, i = it - j * S;
        const int gx = (cx0 - 1) * K + 1 + i, gy = (cy0 - 1) * K + 1 + j;
        const unsigned o = gx >= 1 && gx <= n1 - 2 && gy >= 1 && gy <= n1 - 2
                               ? (unsigned)(gy * n1 + gx) * (unsigned)sizeof(T)
                               : tile2::kOff;
        T v[n], w[n];
#pragma unroll
        for (int z = 0; z < n; ++z) {
          if constexpr (sizeof(T) == 8)
            v[z] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(buf, (int)o, z * ps, 0));
          else
            v[z] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(buf, (int)o, z * ps, 0));
        }
        const T* Q = Qg + scalar(tz * NN);
#pragma unroll
        for (int c = 0; c < n; ++c) w[c] = T(0);
#pragma unroll
        for (int z = 0; z < n; ++z)
#pragma unroll
          for (int c = 0; c < n; ++c) w[c] += Q[z * n + c] * v[z];
#pragma unroll
        for (int c = 0; c < n; ++c) pool[(c * S + j) * MP + i] = w[c];
      }
    }
    __syncthreads();
    // x forward, rows fastest across lanes
    for (int it = t; it < n * S; it += NTH) {
      T* row = pool + it * MP;
      T v[S];
#pragma unroll
      for (int i = 0; i < S; ++i) v[i] = row[i];
#pragma unroll
      for (int s = 0; s < V; ++s) {
        const int vx = cx0 + s;
        T w[n];
#pragma unroll
        for (int c = 0; c < n; ++c) w[c] = T(0);
        if (vx >= 1 && vx <= N - 1) {
          const T* Q = Qg + scalar(variant(vx, N) * NN);
#pragma unroll
          for (int j = 0; j < n; ++j)
#pragma unroll
            for (int c = 0; c < n; ++c) w[c] += Q[j * n + c] * v[s * K + j];
        }
#pragma unroll
        for (int c = 0; c < n; ++c) row[s * n + c] = w[c];
      }
    }
    __syncthreads();
    // y: lines (z mode, x mode), x modes fastest across lanes
    for (int it = t; it < n * M; it += NTH) {
      const int zm = it / M, m = it - zm * M, s = m / n;
      T* line = pool + zm * S * MP + m;
      const T lxz = sLam[variant(min(max(cx0 + s, 1), N - 1), N) * n + m - s * n] + sLam[tz * n + zm];
      T v[S], out[TX];
#pragma unroll
      for (int i = 0; i < S; ++i) v[i] = line[i * MP];
#pragma unroll
      for (int i = 0; i < TX; ++i) out[i] = T(0);
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const int vy = cy0 + u;
        if (vy >= 1 && vy <= N - 1) {
          const int ty = variant(vy, N);
          const T* Q = Qg + scalar(ty * NN);
          T w[n];
#pragma unroll
          for (int c = 0; c < n; ++c) w[c] = T(0);
#pragma unroll
          for (int j = 0; j < n; ++j)
#pragma unroll
            for (int c = 0; c < n; ++c) w[c] += Q[j * n + c] * v[u * K + j];
#pragma unroll
          for (int c = 0; c < n; ++c) w[c] /= lxz + sLam[ty * n + c];
          Q = Qg + scalar(ty * NN);
#pragma unroll
          for (int a = 0; a < n; ++a) {
            const int l = (u - 1) * K + 1 + a;  // owned y node
            if (l >= 0 && l < TX) {  // a sum of its own per patch: one chain would round at the size of the total
              T s1 = T(0);
#pragma unroll
              for (int c = 0; c < n; ++c) s1 += Q[a * n + c] * w[c];
              out[l] += s1;
            }
          }
        }
      }
#pragma unroll
      for (int i = 0; i < TX; ++i) line[i * MP] = out[i];
    }
    __syncthreads();
    // x back
    for (int it = t; it < n * TX; it += NTH) {
      const int zm = it / TX;
      T* row = pool + (zm * S + it - zm * TX) * MP;
      T out[TX];
#pragma unroll
      for (int i = 0; i < TX; ++i) out[i] = T(0);
#pragma unroll
      for (int s = 0; s < V; ++s) {
        const int vx = cx0 + s;
        if (vx >= 1 && vx <= N - 1) {
          const T* Q = Qg + scalar(variant(vx, N) * NN);
          T w[n];
#pragma unroll
          for (int c = 0; c < n; ++c) w[c] = row[s * n + c];
#pragma unroll
          for (int a = 0; a < n; ++a) {
            const int l = (s - 1) * K + 1 + a;
            if (l >= 0 && l < TX) {  // a sum of its own per patch: one chain would round at the size of the total
              T s1 = T(0);
#pragma unroll
              for (int c = 0; c < n; ++c) s1 += Q[a * n + c] * w[c];
              out[l] += s1;
            }
          }
        }
      }
#pragma unroll
      for (int i = 0; i < TX; ++i) row[i] = out[i];
    }
    __syncthreads();
    // z back onto the layer's nodes
    if (t < TX * TX) {
      const T* col = pool + (t / TX) * MP + t % TX;
      T w[n];
#pragma unroll
      for (int c = 0; c < n; ++c) w[c] = col[c * S * MP];
      // the layer's node p is node p + K - 1 of the patch at its lower vertex, p - 1 of the one at its upper vertex
      const T* Q = Qg + scalar(tz * NN);
      if (h == 0) {
#pragma unroll
        for (int p = 0; p < K; ++p)
#pragma unroll
          for (int c = 0; c < n; ++c) acc[p] += Q[(p + K - 1) * n + c] * w[c];
      } else {
#pragma unroll
        for (int p = 1; p < K; ++p)
#pragma unroll
          for (int c = 0; c < n; ++c) acc[p] += Q[(p - 1) * n + c] * w[c];
      }
    }
    __syncthreads();
  }
  if (t < TX * TX) {
    const int gx = cx0 * K + t % TX, gy = cy0 * K + t / TX;
    const size_t g = ((size_t)cz * K * n1 + gy) * n1 + gx;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const bool inner = gx > 0 && gy > 0 && (cz > 0 || p > 0);
      xout[g + p * pl] = inner ? (xin ? xin[g + p * pl] : T(0)) + omega * acc[p] : T(0);
    }
  }
}

template <typename T, int K>
hipError_t patch3d_box_k(int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega, hipStream_t s) {
  using G = PatchBox<K>;
  const int n1 = K * N + 1, nt = N / G::TC, total = nt * nt * N;
  // the planes of a patch are addressed with 31 bits
  if ((2.0 * K - 1) * n1 * n1 * sizeof(T) >= 2147483648.0) return hipErrorInvalidValue;
  patch3d_box_kernel<T, K, G::NTH><<<total + face_blocks<G::NTH>(n1), G::NTH, 0, s>>>(
      r, xin, xout, N, n1, e.Q, e.lam, omega, nt, tile2::magic(nt), total);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_patch3d_box(int k, int N, const LevelEig<T>& e, const T* r, const T* xin, T* xout, T omega,
                              hipStream_t s) {
  switch (k) {
    case 4: return patch3d_box_k<T, 4>(N, e, r, xin, xout, omega, s);
    case 5: return patch3d_box_k<T, 5>(N, e, r, xin, xout, omega, s);
    case 6: return patch3d_box_k<T, 6>(N, e, r, xin, xout, omega, s);
    case 7: return patch3d_box_k<T, 7>(N, e, r, xin, xout, omega, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_patch3d_box<double>(int, int, const LevelEig<double>&, const double*, const double*,
                                               double*, double, hipStream_t);
template hipError_t launch_patch3d_box<float>(int, int, const LevelEig<float>&, const float*, const float*, float*,
                                              float, hipStream_t);

}  // namespace c0ip
