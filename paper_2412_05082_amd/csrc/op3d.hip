// 3D matrix-free C0IP operator for gfx950 (Sec. 4, eq. c0iptensorvp3D
// used on the whole Cartesian mesh).  With the factors listed (z, y, x),
//   A = B M M + M B M + M M B + 2 (L L M + M L L + L M L).
// Grouped by the z factor, with per-plane sums over x and y
//   S1 = M_y (X B_x) + B_y (X M_x) + 2 L_y (X L_x),
//   S2 = M_y (X M_x),
//   S3 = 2 (L_y (X M_x) + M_y (X L_x)),
// the output is Y = M_z S1 + B_z S2 + L_z S3.
//
// Up to degree 4 and from 64^3 cells on (32^3 at k = 2; op3d_box.hip below):
// a workgroup owns a TY x TX column of output nodes (whole cells) over a
// chunk of z cells and streams through the planes of the chunk plus a
// 2k-plane halo on each side:
//   * the plane is staged once in LDS with a 2k-node halo in x and y (the
//     next plane is already on its way from HBM in registers);
//   * one x pass per window of input row computes X M_x, X L_x and X B_x
//     into three LDS buffers;
//   * each thread owns one x column and one cell of y rows, so the y
//     positions in the cell, and with them the band shapes, are known at
//     compile time; the y passes give S1, S2, S3 of its k nodes;
//   * the z factor is applied in scatter form: 1D matrices are symmetric,
//     so plane zs adds row zs of M_z, B_z, L_z times its S values into a
//     register window of the 4k+1 output planes it reaches; the oldest
//     cell of the window is complete after the first plane of each cell
//     and is written out.
// Coefficients: with the default penalty the rows of the periodic classes
// are h-scaled copies of reference rows (h = 1) that are compile-time
// constants (generated at build time by gen_refcoef.cpp); every term of the
// 3D operator then carries the same factor 1/h, applied to the output.
// Along x and y every tile uses these constants: boundary nodes are staged
// as 0, which drops their columns, and in the only other boundary rows, the k
// rows of B next to either end (the point term at the boundary), the lanes
// that own those cells take other constants for the columns that differ.
// Rows of boundary nodes are masked on the way out.  (Redoing every product
// of the boundary tiles with per-lane rows from an LDS table took 441 us
// for 30 % of the tiles of 3D Q3 128^3 in float64, against 337 us for the
// other 70 %, in a launch of its own because of its registers.)  The z
// rows come from the level's reference-scaled table with wave-uniform
// addresses: a plane's row is the same for the whole workgroup.  Output
// nodes on the faces x, y or z = 1 (the last node) are boundary nodes:
// tiles cover nodes [0, kN), and extra workgroups write those faces as
// zeros.
#include <algorithm>
#include <type_traits>

#include "faces3d.h"
#include "kernels.h"
#include "rawbuf.h"
#include "refband.h"
#include "tiles.h"

namespace c0ip {
namespace {

using rawbuf::kOff;
using ref::band_ref;
using tile::Band;

// The coefficient loads of a boundary plane are loop invariant; hoisted
// out of the plane loop they would not fit the scalar registers.  Passing
// the row offset through an empty asm statement on a scalar register keeps
// them inside.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Coefficient of B at column j (a cell's nodes count from 0) of the cell's row p, for rows whose boundary term is at
// the lower end (E = 1), at the upper end (E = 2) or absent (E = 0).
template <int K, int E>
constexpr double edge_b(int p, int j) {
  if (E == 1) return p > 0 ? RefCoef<K>::bl[p - 1][j - 1] : RefCoef<K>::bl[K - 1][K + j - 1];
  if (E == 2) return RefCoef<K>::bl[K - 1 - p][K - 1 - j];
  return RefCoef<K>::b[p][2 * K + j - p];
}

// a += the columns lo..hi of the cell's row p.
template <typename T, int K, int E>
__device__ __forceinline__ T edge_sum(T a, const T* v, int p, int lo, int hi) {
#pragma unroll
  for (int j = lo; j <= hi; ++j) a = ref::mad((T)edge_b<K, E>(p, j), v[j], a);
  return a;
}

// The k rows of B of cell c: a[p] = row p times the input, v[j] = the input at the cell's node j.  The rows next to
// either end differ from the periodic ones in the k coefficients of the boundary cell's nodes only (the point term
// there), so a row is one sum, from its lowest column up, whose columns around its own cell take the coefficients
// that hold there.  (Whole second products for those rows reach three cells, for which the window along z leaves no
// registers: Q3 128^3 float64 spills, 679 us against 418.  The periodic product plus the difference of the
// coefficients rounds at the size of the larger of the two, up to 2.1 times the error of a row at k = 4, and is no
// faster: Q3 128^3 float64 429 us against 424 here, Q2 96 against 88.)  Meshes of at least three cells.
template <typename T, int K>
__device__ __forceinline__ void rows_b(T (&a)[K], const T* v, int c, int N) {
  a[0] = (T)edge_b<K, 0>(0, -2 * K) * v[-2 * K];
  a[0] = edge_sum<T, K, 0>(a[0], v, 0, 1 - 2 * K, -K);
#pragma unroll
  for (int p = 1; p < K; ++p) {
    a[p] = (T)edge_b<K, 0>(p, -K) * v[-K];
    a[p] = edge_sum<T, K, 0>(a[p], v, p, 1 - K, -1);
  }
  if (c > 1 && c < N - 1) {
    a[0] = edge_sum<T, K, 0>(a[0], v, 0, 1 - K, K - 1);
#pragma unroll
    for (int p = 1; p < K; ++p) a[p] = edge_sum<T, K, 0>(a[p], v, p, 0, K);
  } else if (c == N - 1) {  // node k is on the boundary, its value 0
    a[0] = edge_sum<T, K, 0>(a[0], v, 0, 1 - K, -1);
#pragma unroll
    for (int p = 0; p < K; ++p) a[p] = edge_sum<T, K, 2>(a[p], v, p, 0, K - 1);
  } else if (c == 1) {
    a[0] = edge_sum<T, K, 1>(a[0], v, 0, 1 - K, 0);
    a[0] = edge_sum<T, K, 0>(a[0], v, 0, 1, K - 1);
#pragma unroll
    for (int p = 1; p < K; ++p) a[p] = edge_sum<T, K, 0>(a[p], v, p, 0, K);
  } else {  // the first cell: node 0 is on the boundary
#pragma unroll
    for (int p = 1; p < K; ++p) a[p] = edge_sum<T, K, 1>(a[p], v, p, 1, K);
  }
  a[0] = edge_sum<T, K, 0>(a[0], v, 0, K, 2 * K);
#pragma unroll
  for (int p = 1; p < K; ++p) a[p] = edge_sum<T, K, 0>(a[p], v, p, K + 1, 2 * K);
}

// Tile geometry: TXC x TYC cells, x items of CW cells.  One thread per
// (x column, y cell).
template <int K_, int TXC_, int TYC_, int CW_>
struct Geo3 {
  static constexpr int K = K_, TXC = TXC_, TYC = TYC_, CW = CW_;
  static constexpr int H = 2 * K, W = 4 * K + 1, TX = TXC * K, TY = TYC * K, RX = TX + 4 * K, RY = TY + 4 * K;
  // LDS row strides: odd, so that lanes walking down a column hit distinct banks
  static constexpr int RXP = RX | 1, TXP = TX | 1;
  static constexpr int NTH = TX * TYC;
  static constexpr int NXG = TXC / CW, NXI = RY * NXG;
  static constexpr int NST = RX * RY, NL = (NST + NTH - 1) / NTH;
  static_assert(TXC % CW == 0, "x items must divide the tile");
  static_assert(NTH % 64 == 0 && NTH <= 1024, "whole waves");
};

// X M_x on all staged rows, X L_x and X B_x on rows [k, RY - k).  Item
// (row r, group g of CW cells), rows fastest across lanes; cx0 = the tile's
// first cell.
template <typename T, class G>
__device__ __forceinline__ void xpass3(const T* __restrict__ sX, T* __restrict__ sTM, T* __restrict__ sTL,
                                       T* __restrict__ sTB, int cx0, int N) {
  constexpr int K = G::K, CW = G::CW, H = G::H;
  constexpr int LO = Band<2, K>::win_lo(0), HI = Band<2, K>::win_hi() + (CW - 1) * K;
  for (int it = threadIdx.x; it < G::NXI; it += G::NTH) {
    const int g = it / G::RY, r = it - g * G::RY;
    T in[HI - LO + 1];
#pragma unroll
    for (int j = LO; j <= HI; ++j) in[j - LO] = sX[r * G::RXP + g * CW * K + j];
    auto pass = [&](auto opc, T* __restrict__ out) {
      constexpr int OP = decltype(opc)::value;
#pragma unroll
      for (int w = 0; w < CW; ++w) {
        const T* v = in + (w * K + H - LO);
        T a[K];
        if constexpr (OP == 2) {
          rows_b<T, K>(a, v, cx0 + g * CW + w, N);
        } else {
#pragma unroll
          for (int p = 0; p < K; ++p) a[p] = band_ref<T, OP, K>(v + p, p);
        }
#pragma unroll
        for (int p = 0; p < K; ++p) out[(g * CW + w) * K + p] = a[p];
      }
    };
    pass(std::integral_constant<int, 0>{}, sTM + r * G::TXP);
    if (r >= K && r < G::RY - K) {
      pass(std::integral_constant<int, 1>{}, sTL + (r - K) * G::TXP);
      pass(std::integral_constant<int, 2>{}, sTB + (r - K) * G::TXP);
    }
  }
}

// S1, S2, S3 of this thread's k nodes (x column l, y cell cy).  T_B and
// T_L hold staged rows [k, RY - k) (node y0 + cy k + p + o is their row
// cy k + p + k + o), T_M all staged rows (row cy k + p + 2k + o).
template <typename T, class G>
__device__ __forceinline__ void ypass3(const T* __restrict__ sTM, const T* __restrict__ sTL,
                                       const T* __restrict__ sTB, T (&S1)[G::K], T (&S2)[G::K], T (&S3)[G::K],
                                       int cy0, int N) {
  constexpr int K = G::K, TX = G::TX;
  const int l = threadIdx.x % TX, cy = threadIdx.x / TX;
  constexpr int TXP = G::TXP;
  // one window at a time (the scheduling barriers keep the next window's
  // loads from being hoisted over the current one's products)
  {
    T t[3 * K];
#pragma unroll
    for (int j = 0; j < 3 * K; ++j) t[j] = sTB[(cy * K + j) * TXP + l];
#pragma unroll
    for (int p = 0; p < K; ++p) S1[p] = band_ref<T, 0, K>(t + p + K, p);
  }
  __builtin_amdgcn_sched_barrier(0);
  {
    T t[3 * K];
#pragma unroll
    for (int j = 0; j < 3 * K; ++j) t[j] = sTL[(cy * K + j) * TXP + l];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      S1[p] += T(2) * band_ref<T, 1, K>(t + p + K, p);
      S3[p] = band_ref<T, 0, K>(t + p + K, p);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  {
    T t[5 * K];
#pragma unroll
    for (int j = 0; j < 5 * K; ++j) t[j] = sTM[(cy * K + j) * TXP + l];
    T sb[K];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const T* v = t + p + 2 * K;
      S2[p] = band_ref<T, 0, K>(v, p);
      S3[p] = T(2) * (S3[p] + band_ref<T, 1, K>(v, p));
    }
    rows_b<T, K>(sb, t + 2 * K, cy0 + cy, N);
#pragma unroll
    for (int p = 0; p < K; ++p) S1[p] += sb[p];
  }
}

// Plane zs at cell position PS adds row zs of M_z, L_z, B_z (reference
// scaled, read with wave-uniform addresses) times S1, S3, S2 into the
// window: slot j is output plane (c - 2) k + j when zs = c k + PS.
template <typename T, int K, int PS, int OP>
__device__ __forceinline__ void zterm(T (&acc)[4 * K + 1][K], const T (&S)[K], const T* __restrict__ c) {
  constexpr int J = 2 * K + PS;
#pragma unroll
  for (int o = Band<OP, K>::lo(PS); o <= Band<OP, K>::hi(PS); ++o) {
    const T cv = c[o];
#pragma unroll
    for (int p = 0; p < K; ++p) acc[J + o][p] += cv * S[p];
  }
}
template <typename T, int K, int PS>
__device__ __forceinline__ void zscatter(T (&acc)[4 * K + 1][K], const T (&S1)[K], const T (&S2)[K],
                                         const T (&S3)[K], const T* __restrict__ ref, int row, int nclass) {
  constexpr int W = 4 * K + 1, H = 2 * K;
  zterm<T, K, PS, 0>(acc, S1, ref + opaque(row * W + H));
  zterm<T, K, PS, 1>(acc, S3, ref + opaque((nclass + row) * W + H));
  zterm<T, K, PS, 2>(acc, S2, ref + opaque((2 * nclass + row) * W + H));
}

template <typename Tin, typename T, class G, bool RES>
__device__ __forceinline__ void apply3d_tile(const Tin* __restrict__ x, const T* __restrict__ b, T* __restrict__ y,
                                             int N, int n1, const T* __restrict__ ref, T hinv, int nclass, int left,
                                             int right0, int periodic, int cx0, int cy0, int c0, int c1,
                                             T* __restrict__ sX, T* __restrict__ sTM, T* __restrict__ sTL,
                                             T* __restrict__ sTB) {
  constexpr int K = G::K, H = G::H, NL = G::NL, NTH = G::NTH;
  const int NK = n1 - 1, x0 = cx0 * K, y0 = cy0 * K;
  const size_t plane = (size_t)n1 * n1;
  const unsigned pin = (unsigned)(plane * sizeof(Tin)), pout = (unsigned)(plane * sizeof(T));
  const int l = threadIdx.x % G::TX, cy = threadIdx.x / G::TX;
  const int gx = x0 + l;
  // in-plane byte offsets of this thread's staged elements (kOff: boundary or outside)
  unsigned soff[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    const int e = threadIdx.x + q * NTH;
    const int r = e / G::RX, c = e - r * G::RX;
    const int sy = y0 - H + r, sx = x0 - H + c;
    soff[q] = (e < G::NST && sy >= 1 && sy < NK && sx >= 1 && sx < NK) ? (unsigned)(sy * n1 + sx) * sizeof(Tin)
                                                                       : kOff;
  }
  // output offsets (nodes of the tile below kN) and right-hand side offsets
  // (interior nodes only: the residual is 0 on the boundary)
  unsigned yoff[K], boff[K];
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const int gy = y0 + cy * K + p;
    const unsigned o = (unsigned)(gy * n1 + gx) * sizeof(T);
    yoff[p] = gx < NK && gy < NK ? o : kOff;
    boff[p] = gx >= 1 && gx < NK && gy >= 1 && gy < NK ? o : kOff;
  }
  T v[NL];
  // planes that contribute to outputs [c0 k, c1 k), without the boundary planes
  const int zA = max((c0 - 2) * K, 1), zB = min((c1 + 1) * K, NK - 1);
  auto load_plane = [&](int z) {  // zeros beyond plane zB
    const __amdgpu_buffer_rsrc_t r = rawbuf::make(x + (size_t)z * plane, z <= zB ? pin : 0u);
#pragma unroll
    for (int q = 0; q < NL; ++q) v[q] = (T)rawbuf::load<Tin>(r, soff[q]);
  };
  auto store_plane = [&]() {
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int e = threadIdx.x + q * NTH, r = e / G::RX;
      sX[e + r * (G::RXP - G::RX)] = v[q];  // rows padded to RXP; sX also holds the tail of the last q
    }
  };
  T acc[4 * K + 1][K];
#pragma unroll
  for (int j = 0; j <= 4 * K; ++j)
#pragma unroll
    for (int p = 0; p < K; ++p) acc[j][p] = T(0);
  load_plane(zA);
  store_plane();
  load_plane(zA + 1);
  T bq[RES ? K : 1][K];
  for (int c = c0 - 2; c <= c1 + 1; ++c) {
    const int ce = c - 2;  // the cell written after this cell's first plane
    const bool emit_c = ce >= c0 && ce < c1;
    auto load_b = [&]() {  // cell ce; plane 0 is boundary: an empty buffer reads 0
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int gz = ce * K + j;
        const __amdgpu_buffer_rsrc_t r = rawbuf::make(b + (size_t)gz * plane, gz >= 1 && emit_c ? pout : 0u);
#pragma unroll
        for (int p = 0; p < K; ++p) bq[j][p] = rawbuf::load<T>(r, boff[p]);
      }
    };
    static_for<0, K>([&](auto psc) {
      constexpr int ps = decltype(psc)::value;
      if (ps > 0 && c == c1 + 1) return;
      const int zs = c * K + ps;
      if (zs >= zA && zs <= zB) {
        __syncthreads();  // sX holds plane zs; the previous y passes are done
        xpass3<T, G>(sX, sTM, sTL, sTB, cx0, N);
        __syncthreads();
        store_plane();  // plane zs + 1 (unused after zB)
        load_plane(zs + 2);
        T S1[K], S2[K], S3[K];
        ypass3<T, G>(sTM, sTL, sTB, S1, S2, S3, cy0, N);
        const int clz = tile::row_class(zs, n1, K, left, right0, periodic);
        zscatter<T, K, ps>(acc, S1, S2, S3, ref, clz, nclass);
      }
      if (ps == 0 && emit_c) {
        if constexpr (RES) {
          __builtin_amdgcn_sched_barrier(0);  // not before: the windows of the passes need the registers
          load_b();
        }
        // boundary outputs: x = 0 and y = 0 masked; zero columns of the z rows give
        // acc = 0 on plane 0; b reads 0 there
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const __amdgpu_buffer_rsrc_t r = rawbuf::make(y + (size_t)(ce * K + j) * plane, pout);
#pragma unroll
          for (int p = 0; p < K; ++p) {
            const T a = boff[p] == kOff ? T(0) : hinv * acc[j][p];
            rawbuf::store<T>(r, yoff[p], RES ? bq[j][p] - a : a);
          }
        }
      }
    });
#pragma unroll
    for (int j = 0; j <= 3 * K; ++j)
#pragma unroll
      for (int p = 0; p < K; ++p) acc[j][p] = acc[j + K][p];
#pragma unroll
    for (int j = 3 * K + 1; j <= 4 * K; ++j)
#pragma unroll
      for (int p = 0; p < K; ++p) acc[j][p] = T(0);
  }
}

// One workgroup per (tile, z chunk), each XCD walking a contiguous band of
// them (x fastest, then y: neighbouring tiles share halos in that XCD's L2),
// then the workgroups that zero the faces.
// The register bound holds the residual form of Q3 float64 at 3 waves per SIMD
// (170 registers and 2 waves without it: S(x, b) at 128^3 1325 us against
// 1187).  The other degrees and types are left to the compiler: 54 to 100
// registers, or for Q4 float64 all 256, where a bound would spill the window.
template <typename Tin, typename T, class G, bool RES>
__global__ __launch_bounds__(G::NTH, G::K == 3 && sizeof(T) == 8 ? 3 : 1) void apply3d_kernel(
    const Tin* __restrict__ x, const T* __restrict__ b, T* __restrict__ y, int N, int n1, const T* __restrict__ ref,
    T hinv, int nclass, int left, int right0, int periodic, int tx, int ty, int nz, int zcc) {
  const int total = tx * ty * nz, L = blockIdx.x;
  if (L >= total) {
    zero_faces<T, G::NTH>(y, n1, L - total);
    return;
  }
  const int xcd = L & 7, logical = xcd * (total >> 3) + min(xcd, total & 7) + (L >> 3);
  const int bx = logical % tx, rest = logical / tx, by = rest % ty, bz = rest / ty;
  __shared__ T sX[G::NL * G::NTH + (G::NL * G::NTH / G::RX + 1) * (G::RXP - G::RX)];
  __shared__ T sTM[G::RY * G::TXP];
  __shared__ T sTL[(G::RY - 2 * G::K) * G::TXP];
  __shared__ T sTB[(G::RY - 2 * G::K) * G::TXP];
  const int c0 = bz * zcc, c1 = min(c0 + zcc, N);
  apply3d_tile<Tin, T, G, RES>(x, b, y, N, n1, ref, hinv, nclass, left, right0, periodic, bx * G::TXC, by * G::TYC,
                               c0, c1, sX, sTM, sTL, sTB);
}

// Tile configuration per degree (k <= 4; the register window of the z
// factor holds (4k+1) k values per thread).
template <int K> struct Apply3Cfg;
template <> struct Apply3Cfg<2> { using G = Geo3<2, 16, 8, 2>; };
template <> struct Apply3Cfg<3> { using G = Geo3<3, 16, 4, 2>; };
template <> struct Apply3Cfg<4> { using G = Geo3<4, 8, 4, 2>; };

template <typename Tin, typename T, class G>
hipError_t apply3d_g(int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s) {
  const int n1 = G::K * N + 1;
  const int tx = (N + G::TXC - 1) / G::TXC, ty = (N + G::TYC - 1) / G::TYC;
  // z chunks: 1024 workgroups (what the chip holds at 3 waves per SIMD), down
  // to one cell per chunk: a chunk recomputes 3k + 1 halo planes, but below
  // 1024 workgroups the march along z sets the time (3D Q3 32^3 float64, which
  // boxes take now: 63 us at 8 cells per chunk, 43 at 4, 33 at 1).  Twice as
  // many for Q3 float64 from 128^3: there the halos come from HBM once the workgroups of a plane have drifted apart
  // (A x in us, 1024 against 2048: 128^3 453 and 440, 256^3 3993 and 3164). For the others the halo planes cost more
  // up to 128^3 (Q3 64^3 float64 85 and 121; 128^3 Q2 float64 92 and 105, Q3 float32 212 and 242, Q4 float64 1415 and
  // 1595), and 256^3 would gain little (Q2 float64 678 and 663, Q3 float32 1781 and 1698).
  const int target = G::K == 3 && sizeof(T) == 8 && N >= 128 ? 2048 : 1024;
  int zcc = N;
  while (zcc > 1 && (int64_t)tx * ty * ((N + zcc - 1) / zcc) < target) zcc = (zcc + 1) / 2;
  const int nz = (N + zcc - 1) / zcc, grid = tx * ty * nz + face_blocks<G::NTH>(n1);
  if (b)
    apply3d_kernel<Tin, T, G, true><<<grid, G::NTH, 0, s>>>(x, b, y, N, n1, c.ref, c.hinv, c.nclass, c.left,
                                                            c.right0, c.periodic, tx, ty, nz, zcc);
  else
    apply3d_kernel<Tin, T, G, false><<<grid, G::NTH, 0, s>>>(x, b, y, N, n1, c.ref, c.hinv, c.nclass, c.left,
                                                             c.right0, c.periodic, tx, ty, nz, zcc);
  return hipGetLastError();
}

}  // namespace

template <typename Tin, typename T>
hipError_t launch_apply3d(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s) {
  if (!c.ref) return launch_apply3d_wide<Tin, T>(k, N, c, x, b, y, s);  // not the default penalty
  // Small meshes and high degrees on boxes (op3d_box.hip): below 64 cells the march along z, a plane after the
  // other, sets the time (float64, march against boxes, us: Q2 16^3 11.8 against 6.4, 32^3 12.5 against 12.5,
  // 64^3 30 against 54; Q3 16^3 25.6 against 7.5, 32^3 34 against 24, 64^3 82 against 145; Q4 32^3 91 against 52,
  // 64^3 234 against 368); from degree 5 the march's window does not fit the registers (Q5 32^3 with bands
  // in loops 1267 us against 184, 8^3 433 against 11).
  const bool box = k >= 5 || N <= (k == 2 ? 16 : 32);
  // raw buffer offsets, of 4k + 1 planes of the input in a box and of a plane in the march, must stay below 2^31 bytes
  const double plane = (double)(k * N + 1) * (k * N + 1);
  if ((box ? (4.0 * k + 1) * plane * sizeof(Tin) : plane * sizeof(T)) >= 2147483648.0) return hipErrorInvalidValue;
  if (box) return launch_apply3d_box<Tin, T>(k, N, c, x, b, y, s);
  switch (k) {
    case 2: return apply3d_g<Tin, T, Apply3Cfg<2>::G>(N, c, x, b, y, s);
    case 3: return apply3d_g<Tin, T, Apply3Cfg<3>::G>(N, c, x, b, y, s);
    case 4: return apply3d_g<Tin, T, Apply3Cfg<4>::G>(N, c, x, b, y, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_apply3d<double, double>(int, int, const LevelCoef<double>&, const double*,
                                                   const double*, double*, hipStream_t);
template hipError_t launch_apply3d<float, double>(int, int, const LevelCoef<double>&, const float*,
                                                  const double*, double*, hipStream_t);
template hipError_t launch_apply3d<float, float>(int, int, const LevelCoef<float>&, const float*, const float*,
                                                 float*, hipStream_t);

}  // namespace c0ip
