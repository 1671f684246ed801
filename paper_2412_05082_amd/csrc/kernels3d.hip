// 3D matrix-free C0IP operator with coefficient tables, for gfx950: the form
// that every penalty but the default one takes.
//
// Operator (Sec. 4, eq. c0iptensorvp3D, used globally on the Cartesian
// mesh), first factor along x:
//   A = B M M + M B M + M M B + 2 (L L M + M L L + L M L).
// Sum factorisation: x-sweeps X M_x, X L_x, X B_x; y-sweeps give
//   S1 = (B_x M_y + M_x B_y + 2 L_x L_y) X,  S2 = M_x M_y X,
//   S3 = 2 (M_x L_y + L_x M_y) X;
// and Y = M_z S1 + B_z S2 + L_z S3.
// A workgroup owns a 16 x 16 column of (x, y) nodes and streams along z:
// per plane it stages X on the tile plus a 2k halo in LDS, runs the x- and
// y-sweeps, and pushes S1, S2, S3 of its own column into register windows
// of 4k+1 planes, from which the z-sweep emits one output plane.
#include "kernels.h"

namespace c0ip {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ int row_class(int g, int n1, int k, int left, int right0, int periodic) {
  if (!periodic) return g;
  if (g < left) return g;
  if (g >= right0) return left + (n1 - 1 - g);
  return 2 * left + g % k;
}

template <int K> __host__ __device__ constexpr int m_lo(int p) { return p == 0 ? -K : -p; }
template <int K> __host__ __device__ constexpr int m_hi(int p) { return p == 0 ? K : K - p; }
template <int K> __host__ __device__ constexpr int b_lo(int p) { return p == 0 ? -2 * K : -K - p; }
template <int K> __host__ __device__ constexpr int b_hi(int p) { return p == 0 ? 2 * K : 2 * K - p; }
template <int K> __host__ __device__ constexpr int tab_max() { return 3 * (5 * K + 2) * (4 * K + 1); }

// ------------------------------------------------------------------ operator

constexpr int kT3 = 16;  // tile width in x and y (nodes)

template <typename Tin, typename T, int K, bool RES>
__global__ __launch_bounds__(kThreads) void apply3d_kernel(const Tin* __restrict__ x, const T* __restrict__ b,
                                                           T* __restrict__ y, int n1, int zc,
                                                           const T* __restrict__ tab, int nclass, int left,
                                                           int right0, int periodic) {
  constexpr int H = 2 * K, W = 4 * K + 1, R = kT3 + 2 * H;  // staged plane is R x R
  constexpr int NL = (R * R + kThreads - 1) / kThreads;
  __shared__ T sX[R * R];
  __shared__ T sM[R * kT3];              // X M_x on rows [-2k, T+2k)
  __shared__ T sL[(kT3 + 2 * K) * kT3];  // X L_x on rows [-k, T+k)
  __shared__ T sB[(kT3 + 2 * K) * kT3];  // X B_x on rows [-k, T+k)
  __shared__ T sTab[tab_max<K>()];
  const int x0 = blockIdx.x * kT3, y0 = blockIdx.y * kT3, z0 = blockIdx.z * zc;
  const int ntab = 3 * nclass * W;
  for (int e = threadIdx.x; e < ntab; e += kThreads) sTab[e] = tab[e];
  const int lx = threadIdx.x % kT3, ly = threadIdx.x / kT3;
  const int gx = x0 + lx, gy = y0 + ly;
  const int cy = row_class(min(gy, n1 - 1), n1, K, left, right0, periodic), py = min(gy, n1 - 1) % K;
  T w1[W], w2[W], w3[W];  // S1, S2, S3 at planes zp-4k .. zp
#pragma unroll
  for (int q = 0; q < W; ++q) w1[q] = w2[q] = w3[q] = T(0);
  const size_t plane = (size_t)n1 * n1;
  const int zend = min(z0 + zc, n1);
  for (int zp = z0 - H; zp < zend + H; ++zp) {
    // stage X on the plane (0 outside the mesh)
    {
      T v[NL];
      const bool zin = zp >= 0 && zp < n1;
#pragma unroll
      for (int q = 0; q < NL; ++q) {
        const int e = threadIdx.x + q * kThreads;
        const int r = e / R, c = e - r * R;
        const int yy = y0 - H + r, xx = x0 - H + c;
        v[q] = (e < R * R && zin && yy >= 0 && yy < n1 && xx >= 0 && xx < n1)
                   ? (T)x[(size_t)zp * plane + (size_t)yy * n1 + xx]
                   : T(0);
      }
      __syncthreads();  // previous plane's sweeps are done with sX, sM, sL, sB
#pragma unroll
      for (int q = 0; q < NL; ++q) {
        const int e = threadIdx.x + q * kThreads;
        if (e < R * R) sX[e] = v[q];
      }
    }
    __syncthreads();
    // x-sweeps: item (row r in [0, R), column l in [0, T))
    for (int it = threadIdx.x; it < R * kT3; it += kThreads) {
      const int r = it / kT3, l = it - r * kT3;
      const int g = min(x0 + l, n1 - 1);
      const int cls = row_class(g, n1, K, left, right0, periodic), p = g % K;
      const T* cM = sTab + cls * W + H;
      const T* cL = sTab + (nclass + cls) * W + H;
      const T* cB = sTab + (2 * nclass + cls) * W + H;
      const T* row = sX + r * R + l + H;  // row[o] = X at column x0 + l + o
      T m = 0;
      for (int o = m_lo<K>(p); o <= m_hi<K>(p); ++o) m += cM[o] * row[o];
      sM[it] = m;
      if (r >= K && r < R - K) {
        T lv = 0, bv = 0;
        for (int o = m_lo<K>(p); o <= m_hi<K>(p); ++o) lv += cL[o] * row[o];
        for (int o = b_lo<K>(p); o <= b_hi<K>(p); ++o) bv += cB[o] * row[o];
        sL[(r - K) * kT3 + l] = lv;
        sB[(r - K) * kT3 + l] = bv;
      }
    }
    __syncthreads();
    // y-sweeps for this thread's column
    T s1, s2, s3;
    {
      const T* cM = sTab + cy * W + H;
      const T* cL = sTab + (nclass + cy) * W + H;
      const T* cB = sTab + (2 * nclass + cy) * W + H;
      T bm = 0, mb = 0, mm = 0, ml = 0, ll = 0, lm = 0;
      for (int o = m_lo<K>(py); o <= m_hi<K>(py); ++o) {
        const T xm = sM[(ly + H + o) * kT3 + lx], xl = sL[(ly + K + o) * kT3 + lx],
                xb = sB[(ly + K + o) * kT3 + lx];
        bm += cM[o] * xb;
        mm += cM[o] * xm;
        ml += cL[o] * xm;
        ll += cL[o] * xl;
        lm += cM[o] * xl;
      }
      for (int o = b_lo<K>(py); o <= b_hi<K>(py); ++o) mb += cB[o] * sM[(ly + H + o) * kT3 + lx];
      s1 = bm + mb + 2 * ll;
      s2 = mm;
      s3 = 2 * (ml + lm);
    }
#pragma unroll
    for (int q = 0; q < W - 1; ++q) {
      w1[q] = w1[q + 1];
      w2[q] = w2[q + 1];
      w3[q] = w3[q + 1];
    }
    w1[W - 1] = s1;
    w2[W - 1] = s2;
    w3[W - 1] = s3;
    // z-sweep for plane z = zp - 2k: window index 2k + o holds plane z + o
    const int z = zp - H;
    if (z >= z0 && z < zend && gx < n1 && gy < n1) {
      const int cz = row_class(z, n1, K, left, right0, periodic), pz = z % K;
      const T* cM = sTab + cz * W + H;
      const T* cL = sTab + (nclass + cz) * W + H;
      const T* cB = sTab + (2 * nclass + cz) * W + H;
      T acc = 0;
      for (int o = m_lo<K>(pz); o <= m_hi<K>(pz); ++o) acc += cM[o] * w1[H + o] + cL[o] * w3[H + o];
      for (int o = b_lo<K>(pz); o <= b_hi<K>(pz); ++o) acc += cB[o] * w2[H + o];
      const size_t idx = (size_t)z * plane + (size_t)gy * n1 + gx;
      if (RES) {
        const bool bnd = gx == 0 || gx == n1 - 1 || gy == 0 || gy == n1 - 1 || z == 0 || z == n1 - 1;
        y[idx] = bnd ? T(0) : b[idx] - acc;
      } else {
        y[idx] = acc;
      }
    }
  }
}

template <typename Tin, typename T, int K>
hipError_t apply3d_k(int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s) {
  const int n1 = K * N + 1;
  const int nt = (n1 + kT3 - 1) / kT3;
  // split z so that the grid has a few thousand workgroups; halo planes are recomputed
  int zc = n1;
  while (zc > 8 * K && (int64_t)nt * nt * ((n1 + zc - 1) / zc) < 2048) zc = (zc + 1) / 2;
  dim3 grid(nt, nt, (n1 + zc - 1) / zc);
  if (b)
    apply3d_kernel<Tin, T, K, true><<<grid, kThreads, 0, s>>>(x, b, y, n1, zc, c.tab, c.nclass, c.left, c.right0,
                                                               c.periodic);
  else
    apply3d_kernel<Tin, T, K, false><<<grid, kThreads, 0, s>>>(x, b, y, n1, zc, c.tab, c.nclass, c.left,
                                                                c.right0, c.periodic);
  return hipGetLastError();
}

}  // namespace

template <typename Tin, typename T>
hipError_t launch_apply3d_wide(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s) {
#define CALL(K) apply3d_k<Tin, T, K>(N, c, x, b, y, s)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

template hipError_t launch_apply3d_wide<double, double>(int, int, const LevelCoef<double>&, const double*,
                                                   const double*, double*, hipStream_t);
template hipError_t launch_apply3d_wide<float, double>(int, int, const LevelCoef<double>&, const float*,
                                                  const double*, double*, hipStream_t);
template hipError_t launch_apply3d_wide<float, float>(int, int, const LevelCoef<float>&, const float*, const float*,
                                                 float*, hipStream_t);
}  // namespace c0ip
