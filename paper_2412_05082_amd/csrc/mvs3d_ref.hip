// One colour of the 3D coloured multiplicative smoother (numbering:
// mvs3d.hip) for the default penalty, residual included, in place:
//   x <- x + omega * sum_{v of the colour} R_v^T A~_v^{-1} R_v (b - A x).
// A separate residual pass computes all of b - A x although a colour's
// patches hold a fifth of its nodes, and on a coarse mesh its z march is one
// long serial chain in a few workgroups (11 us at 8^3 to 32^3; 6 us on boxes).
//
// A workgroup owns P consecutive patches of one row of the colour (same vy,
// vz, 4 cells apart in x).  In the grouped form of the operator,
//   A x = M_z U1 + L_z U2 + B_z U3,  U1 = M_y (X B_x) + B_y (X M_x) + 2 L_y (X L_x),
//   U2 = 2 (L_y (X M_x) + M_y (X L_x)),  U3 = M_y (X M_x),
// only B reaches beyond the patch's closed cells: the residual on a patch
// takes the (2k+1)^2 closed x rows (M, L and B) and, k nodes further in y or
// in z, rows that need M alone.  One x pass, one y pass and one z pass with
// compile-time coefficients; the z pass ends in the forward z transform of
// the local solve, whose other transforms run line by line in registers.
//
// One step (16 colours) against a residual pass and a launch of local solves
// per colour: Q2 128^3 float32 1623 -> 1100 us, Q2 8^3 268 -> 82; it is bound
// by instruction issue and, on the finest meshes, by reading x about 1.5 times
// per colour.
//
// Why in place is safe: patches of one colour lie 4 cells apart along an
// axis or 2 along two, so no node that a patch's residual depends on is an
// interior node of another one; what is staged beyond them is not used.
#include <type_traits>

#include "mvs3d.h"
#include "tile2d.h"

namespace c0ip {
namespace {

using ref::band_ref;
using tile::variant;

// P patches on NTH threads, by a sweep: about an item of each part of the x pass and of the y pass per thread. Where P
// does not divide a row of the colour (N / 4 patches) its last workgroup is partly idle. Q2 128^3 float32, us a step:
// P = 6 1100, 4 1265, 8 1233 (384 threads), 3 1393; float64 P = 4 2130, 6 2650; Q3 64^3 float32 P = 2 593, 1 663,
// 3 750; Q4 32^3 P = 1 316, 2 322.
template <int K, int ES> struct Shape3;  // degree, bytes per value
template <int ES> struct Shape3<2, ES> { static constexpr int P = ES == 4 ? 6 : 4, NTH = 256; };
template <int ES> struct Shape3<3, ES> { static constexpr int P = 2, NTH = 256; };
template <int ES> struct Shape3<4, ES> { static constexpr int P = 1, NTH = 256; };

template <int K, int ES>
struct G3 {
  static constexpr int P = Shape3<K, ES>::P, NTH = Shape3<K, ES>::NTH;
  static constexpr int n = 2 * K - 1, NN = n * n, C = 2 * K + 1, W = 4 * K + 1, E = 2 * K;
  static constexpr int WX = 4 * K * P + 1, WXP = WX | 1;  // staged columns, odd LDS stride
  // rows: the closed planes' W rows each, then the outside planes' C closed rows each
  static constexpr int NR = C * W + E * C;
  static constexpr int COL = P * n, TS = COL | 1;         // interior columns, odd LDS stride
  static constexpr int RPI = NTH / WX, SC = (W + RPI - 1) / RPI, SE = (C + RPI - 1) / RPI;  // rows a step, steps
  static constexpr int SZT = (NR + 2 * C * C) * TS;       // X M_x (all rows), X L_x, X B_x (closed rows)
  static constexpr int SZU = (2 * C + W) * n * TS;        // U1, U2, U3 (over the staged x)
  static constexpr int SZX = NR * WXP > SZU ? NR * WXP : SZU;
  static constexpr int XC = C * C * P, XE = 2 * C * E * P;  // x items: closed, outside
  static constexpr int YC = C * COL, YE = E * COL;          // y items
  static_assert(COL * n <= NTH, "a z item per thread");
  static_assert(n * n * TS <= SZT, "the local solve's values go over X M_x");
};

// interior rows of a factor on a patch; v[0] = first node of the closed patch
template <typename T, int OP, int K>
__device__ __forceinline__ void patch_band(const T* v, T (&o)[2 * K - 1]) {
#pragma unroll
  for (int p = 1; p < K; ++p) o[p - 1] = band_ref<T, OP, K>(v + p, p);
#pragma unroll
  for (int p = 0; p < K; ++p) o[K - 1 + p] = band_ref<T, OP, K>(v + K + p, p);
}
// rows of B at vertex v along the axis; w[K] = first node of the window (k nodes before the closed patch; the
// K values before it are never used: they belong to the first cell's row 0)
template <typename T, int K>
__device__ __forceinline__ void patch_b(const T* w, T (&o)[2 * K - 1], int v, int N) {
  T a[K], c[K];
  a[0] = T(0);
#pragma unroll
  for (int p = 1; p < K; ++p) a[p] = band_ref<T, 2, K>(w + 2 * K + p, p);
  ref::boundary_b<T, K>(a, w + 2 * K, v - 1, N);
#pragma unroll
  for (int p = 0; p < K; ++p) c[p] = band_ref<T, 2, K>(w + 3 * K + p, p);
  ref::boundary_b<T, K>(c, w + 3 * K, v, N);
#pragma unroll
  for (int p = 1; p < K; ++p) o[p - 1] = a[p];
#pragma unroll
  for (int p = 0; p < K; ++p) o[K - 1 + p] = c[p];
}

template <typename T, int K, int NTH, bool RES>
__global__ __launch_bounds__(NTH) void mvs3d_colour_ref_kernel(
    const T* __restrict__ b, T* __restrict__ x, int N, int n1, int colour, int nxc, unsigned mx, int nb, unsigned mb, T scale,
    const T* __restrict__ Qg, const T* __restrict__ lamg, T omega) {
  using G = G3<K, sizeof(T)>;
  constexpr int P = G::P, n = G::n, NN = G::NN, C = G::C, W = G::W, E = G::E, TS = G::TS, NR = G::NR;
  __shared__ T sX[RES ? G::SZX : 1];
  __shared__ T sT[RES ? G::SZT : NN * TS];
  __shared__ T sQ[4 * NN];
  __shared__ T sLam[4 * n];
  const int t = threadIdx.x;
  // this workgroup's row of the colour and its patches there
  const unsigned q = tile2::xcd_order(blockIdx.x, gridDim.x), yz = tile2::quotient(q, mx), cb = tile2::quotient(yz, mb);
  const int px = colour & 1, py = (colour >> 1) & 1, pz = (colour >> 2) & 1;
  const Lat la = lat(N, px);
  const int lb = lat(N, py).lo + (int)(yz - cb * nb), lc = lat(N, pz).lo + (int)cb;
  const int par = ((((colour >> 3) & 1) - lc - lb) % 2 + 2) % 2;
  const int af = la.lo + (la.lo + par) % 2 + 2 * P * (int)(q - yz * nxc);
  if (af > la.hi) return;
  const int np = min(P, (la.hi - af) / 2 + 1);
  const int vx0 = 2 * af + px, vy = 2 * lb + py, vz = 2 * lc + pz;
  const int ty = variant(vy, N), tz = variant(vz, N);
  const size_t pl = (size_t)n1 * n1;
  // this thread's z item: interior row zy and column (patch zp, zx)
  const int zy = t / G::COL, zc = t - zy * G::COL, zp = zc / n, zx = zc - zp * n;
  const bool zon = zy < n && zp < np;
  const size_t g0 = ((size_t)((vz - 1) * K + 1) * n1 + (vy - 1) * K + 1 + zy) * n1 + (vx0 + 4 * zp - 1) * K + 1 + zx;
  constexpr int LQ = (4 * NN + NTH - 1) / NTH;
  T qv[LQ], bv[n], xv[n];
#pragma unroll
  for (int u = 0; u < LQ; ++u) qv[u] = t + u * NTH < 4 * NN ? Qg[t + u * NTH] : T(0);
  const T lv = t < 4 * n ? lamg[t] : T(0);
  if (zon) {
#pragma unroll
    for (int z = 0; z < n; ++z) {
      bv[z] = b[g0 + z * pl];
      xv[z] = x[g0 + z * pl];
    }
  }
  if constexpr (RES) {
    // stage x, 0 on and outside the boundary: a thread keeps its column and its rows of a plane, a plane's
    // offset is scalar
    const int r0 = t / G::WX, c0 = t - r0 * G::WX;
    const int gx = (vx0 - 2) * K + c0, zlo = max((vz - 2) * K, 0);
    const bool con = r0 < G::RPI && gx >= 1 && gx <= n1 - 2;
    const int ps = (int)(pl * sizeof(T));
    const __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc(
        x + zlo * pl, (short)0, (min((vz + 2) * K + 1, n1) - zlo) * ps, 0x00020000);
    auto offset = [&](int yy) {
      const int gy = (vy - 2) * K + yy;
      return con && gy >= 1 && gy <= n1 - 2 ? (unsigned)(gy * n1 + gx) * (unsigned)sizeof(T) : tile2::kOff;
    };
    auto load = [&](unsigned o, int zz) {
      const int gz = (vz - 2) * K + zz;
      const bool on = gz >= 1 && gz <= n1 - 2;
      const int so = on ? (gz - zlo) * ps : 0;
      if (!on) o = tile2::kOff;
      if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(buf, (int)o, so, 0));
      else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(buf, (int)o, so, 0));
    };
    T v[C][G::SC], w[E][G::SE];
#pragma unroll
    for (int u = 0; u < G::SC; ++u) {
      const unsigned o = offset(r0 + u * G::RPI);
#pragma unroll
      for (int z = 0; z < C; ++z) v[z][u] = load(o, K + z);
    }
#pragma unroll
    for (int u = 0; u < G::SE; ++u) {
      const unsigned o = offset(K + r0 + u * G::RPI);
#pragma unroll
      for (int e = 0; e < E; ++e) w[e][u] = load(o, e < K ? e : e + C);
    }
    T* s = sX + r0 * G::WXP + c0;
    if (r0 < G::RPI) {
#pragma unroll
      for (int u = 0; u < G::SC; ++u)
        if (W % G::RPI == 0 || u + 1 < G::SC || r0 + u * G::RPI < W) {
#pragma unroll
          for (int z = 0; z < C; ++z) s[(z * W + u * G::RPI) * G::WXP] = v[z][u];
        }
#pragma unroll
      for (int u = 0; u < G::SE; ++u)
        if (C % G::RPI == 0 || u + 1 < G::SE || r0 + u * G::RPI < C) {
#pragma unroll
          for (int e = 0; e < E; ++e) s[(C * W + e * C + u * G::RPI) * G::WXP] = w[e][u];
        }
    }
  }
#pragma unroll
  for (int u = 0; u < LQ; ++u)
    if (t + u * NTH < 4 * NN) sQ[t + u * NTH] = qv[u];
  if (t < 4 * n) sLam[t] = lv;
  __syncthreads();
  T* sTL = sT + NR * TS;
  T* sTB = sTL + C * C * TS;
  T* sU1 = sX;
  T* sU2 = sU1 + C * n * TS;
  T* sU3 = sU2 + C * n * TS;
  if constexpr (RES) {
    // x pass, rows fastest across lanes
    for (int it = t; it < G::XC; it += NTH) {
      const int p = it / (C * C), rc = it - p * (C * C), zi = rc / C, r = zi * W + K + rc - zi * C;
      T in[5 * K + 1], o[n];
#pragma unroll
      for (int j = 0; j < K; ++j) in[j] = T(0);
#pragma unroll
      for (int j = 0; j < W; ++j) in[K + j] = sX[r * G::WXP + p * 4 * K + j];
      patch_band<T, 0, K>(in + 2 * K, o);
#pragma unroll
      for (int j = 0; j < n; ++j) sT[r * TS + p * n + j] = o[j];
      patch_band<T, 1, K>(in + 2 * K, o);
#pragma unroll
      for (int j = 0; j < n; ++j) sTL[rc * TS + p * n + j] = o[j];
      patch_b<T, K>(in, o, vx0 + 4 * p, N);
#pragma unroll
      for (int j = 0; j < n; ++j) sTB[rc * TS + p * n + j] = o[j];
    }
    for (int it = t; it < G::XE; it += NTH) {
      const int p = it / (2 * C * E), re = it - p * (2 * C * E), zi = re / E, out = re - zi * E;
      const int r = re < C * E ? zi * W + (out < K ? out : out + C) : C * W + re - C * E;
      T in[C], o[n];
#pragma unroll
      for (int j = 0; j < C; ++j) in[j] = sX[r * G::WXP + p * 4 * K + K + j];
      patch_band<T, 0, K>(in, o);
#pragma unroll
      for (int j = 0; j < n; ++j) sT[r * TS + p * n + j] = o[j];
    }
    __syncthreads();
    // y pass, columns fastest across lanes; planes outside the closed patch need U3 alone
    constexpr int Y0 = (G::YC + 63) / 64 * 64;  // whole waves
    for (int it = t; it < Y0 + G::YE; it += NTH) {
      if (it < G::YC) {
        const int z = it / G::COL, c = it - z * G::COL;
        T m[5 * K + 1], l[C], a[n], u1[n], u2[n];
#pragma unroll
        for (int j = 0; j < K; ++j) m[j] = T(0);
#pragma unroll
        for (int j = 0; j < W; ++j) m[K + j] = sT[(z * W + j) * TS + c];
        patch_band<T, 0, K>(m + 2 * K, a);
#pragma unroll
        for (int j = 0; j < n; ++j) sU3[((z + K) * n + j) * TS + c] = a[j];
        patch_band<T, 1, K>(m + 2 * K, u2);
        patch_b<T, K>(m, u1, vy, N);
#pragma unroll
        for (int j = 0; j < C; ++j) l[j] = sTL[(z * C + j) * TS + c];
        patch_band<T, 0, K>(l, a);
#pragma unroll
        for (int j = 0; j < n; ++j) sU2[(z * n + j) * TS + c] = T(2) * (u2[j] + a[j]);
        patch_band<T, 1, K>(l, a);
#pragma unroll
        for (int j = 0; j < n; ++j) u1[j] += T(2) * a[j];
#pragma unroll
        for (int j = 0; j < C; ++j) l[j] = sTB[(z * C + j) * TS + c];
        patch_band<T, 0, K>(l, a);
#pragma unroll
        for (int j = 0; j < n; ++j) sU1[(z * n + j) * TS + c] = u1[j] + a[j];
      } else if (it >= Y0) {
        const int e = (it - Y0) / G::COL, c = it - Y0 - e * G::COL;
        T m[C], a[n];
#pragma unroll
        for (int j = 0; j < C; ++j) m[j] = sT[(C * W + e * C + j) * TS + c];
        patch_band<T, 0, K>(m, a);
#pragma unroll
        for (int j = 0; j < n; ++j) sU3[((e < K ? e : e + C) * n + j) * TS + c] = a[j];
      }
    }
    __syncthreads();
  }
  // z pass, then the forward z transform
  T* sR = sT;
  const T* qz = sQ + tz * NN;
  const T* qy = sQ + ty * NN;
  if (zy < n) {
    T r[n];
    if constexpr (RES) {
      T m[5 * K + 1], a[n];
#pragma unroll
      for (int j = 0; j < K; ++j) m[j] = T(0);
#pragma unroll
      for (int j = 0; j < W; ++j) m[K + j] = sU3[(j * n + zy) * TS + zc];
      patch_b<T, K>(m, r, vz, N);
#pragma unroll
      for (int j = 0; j < C; ++j) m[j] = sU1[(j * n + zy) * TS + zc];
      patch_band<T, 0, K>(m, a);
#pragma unroll
      for (int j = 0; j < n; ++j) r[j] += a[j];
#pragma unroll
      for (int j = 0; j < C; ++j) m[j] = sU2[(j * n + zy) * TS + zc];
      patch_band<T, 1, K>(m, a);
#pragma unroll
      for (int j = 0; j < n; ++j) r[j] = zon ? bv[j] - scale * (r[j] + a[j]) : T(0);
    } else {
#pragma unroll
      for (int j = 0; j < n; ++j) r[j] = zon ? bv[j] : T(0);
    }
#pragma unroll
    for (int c = 0; c < n; ++c) {
      T s = 0;
#pragma unroll
      for (int z = 0; z < n; ++z) s += qz[z * n + c] * r[z];
      sR[(c * n + zy) * TS + zc] = s;
    }
  }
  __syncthreads();
  // y lines, in place
  auto ylines = [&](auto fwd) {
    for (int it = t; it < n * G::COL; it += NTH) {
      const int z = it / G::COL;
      T* s = sR + z * n * TS + it - z * G::COL;
      T v[n];
#pragma unroll
      for (int j = 0; j < n; ++j) v[j] = s[j * TS];
#pragma unroll
      for (int c = 0; c < n; ++c) {
        T a = 0;
#pragma unroll
        for (int j = 0; j < n; ++j) a += (decltype(fwd)::value ? qy[j * n + c] : qy[c * n + j]) * v[j];
        s[c * TS] = a;
      }
    }
    __syncthreads();
  };
  ylines(std::true_type{});
  // x lines: forward, reciprocal eigenvalue sums, back
  for (int it = t; it < NN * P; it += NTH) {
    const int p = it / NN, line = it - p * NN, z = line / n, y = line - z * n;
    const int tx = variant(min(vx0 + 4 * p, N - 1), N);
    const T* qx = sQ + tx * NN;
    const T lyz = sLam[ty * n + y] + sLam[tz * n + z];
    T* s = sR + line * TS + p * n;
    T v[n], w[n];
#pragma unroll
    for (int j = 0; j < n; ++j) v[j] = s[j];
#pragma unroll
    for (int c = 0; c < n; ++c) {
      T a = 0;
#pragma unroll
      for (int j = 0; j < n; ++j) a += qx[j * n + c] * v[j];
      w[c] = a / (sLam[tx * n + c] + lyz);
    }
#pragma unroll
    for (int c = 0; c < n; ++c) {
      T a = 0;
#pragma unroll
      for (int j = 0; j < n; ++j) a += qx[c * n + j] * w[j];
      s[c] = a;
    }
  }
  __syncthreads();
  ylines(std::false_type{});
  if (zon) {
    T v[n];
#pragma unroll
    for (int j = 0; j < n; ++j) v[j] = sR[(j * n + zy) * TS + zc];
#pragma unroll
    for (int c = 0; c < n; ++c) {
      T a = 0;
#pragma unroll
      for (int j = 0; j < n; ++j) a += qz[c * n + j] * v[j];
      x[g0 + c * pl] = xv[c] + omega * a;
    }
  }
}

template <typename T, int K>
hipError_t mvs3d_ref_k(int N, int colour, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b, const T* r, T* x,
                       T omega, hipStream_t s) {
  using G = G3<K, sizeof(T)>;
  const Lat a = lat(N, colour & 1), bb = lat(N, (colour >> 1) & 1), cc = lat(N, (colour >> 2) & 1);
  const int nb = bb.hi - bb.lo + 1, nc = cc.hi - cc.lo + 1, na = (a.hi - a.lo) / 2 + 1;
  if (a.hi < a.lo || nb <= 0 || nc <= 0) return hipSuccess;
  const int nxc = (na + G::P - 1) / G::P, total = nxc * nb * nc;
  const unsigned mx = tile2::magic(nxc), mb = tile2::magic(nb);
  if (r)
    mvs3d_colour_ref_kernel<T, K, G::NTH, false><<<total, G::NTH, 0, s>>>(r, x, N, K * N + 1, colour, nxc, mx, nb, mb,
                                                                     c.hinv, e.Q, e.lam, omega);
  else
    mvs3d_colour_ref_kernel<T, K, G::NTH, true><<<total, G::NTH, 0, s>>>(b, x, N, K * N + 1, colour, nxc, mx, nb, mb,
                                                                    c.hinv, e.Q, e.lam, omega);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_mvs3d_colour_ref(int k, int N, int colour, const LevelCoef<T>& c, const LevelEig<T>& e, const T* b,
                                   const T* r, T* x, T omega, hipStream_t s) {
  switch (k) {
    case 2: return mvs3d_ref_k<T, 2>(N, colour, c, e, b, r, x, omega, s);
    case 3: return mvs3d_ref_k<T, 3>(N, colour, c, e, b, r, x, omega, s);
    case 4: return mvs3d_ref_k<T, 4>(N, colour, c, e, b, r, x, omega, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_mvs3d_colour_ref<double>(int, int, int, const LevelCoef<double>&, const LevelEig<double>&,
                                                    const double*, const double*, double*, double, hipStream_t);
template hipError_t launch_mvs3d_colour_ref<float>(int, int, int, const LevelCoef<float>&, const LevelEig<float>&,
                                                   const float*, const float*, float*, float, hipStream_t);

}  // namespace c0ip
