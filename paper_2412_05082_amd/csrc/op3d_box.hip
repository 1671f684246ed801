// 3D C0IP operator on boxes of cells (default penalty): same result as
// op3d.hip, without its march along z.  Grouped by the x and y factors,
//   A x = M_y V1 + L_y V2 + B_y V3,  V1 = (M_z X) B_x + (B_z X) M_x + 2 (L_z X) L_x,
//   V2 = 2 ((M_z X) L_x + (L_z X) M_x),  V3 = (M_z X) M_x.
// A workgroup owns TC x TC cells of one cell layer.  One thread per column of
// the box reads its 4k + 1 planes and writes M_z X, L_z X and B_z X of the
// layer's k planes to LDS (L and B on the closed cells only: nothing else
// needs them); an x pass per (row, cell) and a y pass per (column, cell), each
// over all k planes at once, finish.  Three phases instead of a chain of 5k
// or more planes, each with two barriers and a load to wait for, and no
// accumulators: the march holds (4k+1) k of them per thread, which only fits
// up to k = 4.  Small meshes are bound by the latency of the three phases (Q5
// 4^3 float64 429 -> 11 us, Q3 16^3 57 -> 7.5), large ones by instruction
// issue (at Q5 32^3 float64 vector instructions take 40 % of the SIMDs' slots,
// with nearly as many scalar ones beside them: 1267 -> 184 us, Q7 32^3 5084 ->
// 630), most of it for the columns that neighbouring boxes recompute.
#include <type_traits>

#include "faces3d.h"
#include "kernels.h"
#include "tile2d.h"

namespace c0ip {
namespace {

using ref::band_ref;

template <int K> struct BoxThreads;  // an x item per thread (the x pass writes over its own input), whole waves
template <> struct BoxThreads<2> { static constexpr int NTH = 64; };
template <> struct BoxThreads<3> { static constexpr int NTH = 128; };
template <> struct BoxThreads<4> { static constexpr int NTH = 192; };
template <> struct BoxThreads<5> { static constexpr int NTH = 320; };
template <> struct BoxThreads<6> { static constexpr int NTH = 448; };
template <> struct BoxThreads<7> { static constexpr int NTH = 576; };

template <int K_>
struct Box {
  static constexpr int K = K_, TC = 2, NTH = BoxThreads<K>::NTH, TX = TC * K;
  static constexpr int C = 2 * K + 1, W = 4 * K + 1, E = 2 * K;   // closed and whole 1D windows; rows outside
  static constexpr int RX = (TC + 3) * K + 1, RC = (TC + 1) * K + 1;  // columns of the box; on the closed cells
  // LDS row strides: odd, so that lanes walking down the rows hit distinct banks
  static constexpr int RXP = RX | 1, RCP = RC | 1, TXP = TX | 1;
  static constexpr int SM = RC * RXP + E * RCP, SC = RC * RCP;  // M_z X (no corners), L_z X or B_z X of a plane
  static constexpr int SV = (RX + 2 * RC) * TXP;                // V3, V1, V2 of a plane
  static constexpr int SZ = K * (SM + 2 * SC > SV ? SM + 2 * SC : SV);
  static constexpr int NZ = RC * RX + E * RC;                   // columns without the corners
  static constexpr int XC = K * RC * TC, XE = K * E * TC, NY = K * TX * TC;
  static_assert(XC <= NTH && XE <= NTH, "an x item of each kind per thread at most");
};

template <typename Tin, typename T, int K, int NTH, bool RES>
__global__ __launch_bounds__(NTH) void apply3d_box_kernel(const Tin* __restrict__ x, const T* __restrict__ b,
                                                          T* __restrict__ y, int N, int n1, T scale, int nt,
                                                          unsigned mt, int total) {
  using G = Box<K>;
  constexpr int TC = G::TC, TX = G::TX, C = G::C, W = G::W, E = G::E, RX = G::RX, RC = G::RC, RXP = G::RXP,
                RCP = G::RCP, TXP = G::TXP;
  if ((int)blockIdx.x >= total) {
    zero_faces<T, NTH>(y, n1, blockIdx.x - total);
    return;
  }
  __shared__ T pool[G::SZ];
  const unsigned q = tile2::xcd_order(blockIdx.x, total), yz = tile2::quotient(q, mt), cz_ = tile2::quotient(yz, mt);
  const int cx0 = (int)(q - yz * nt) * TC, cy0 = (int)(yz - cz_ * nt) * TC, cz = (int)cz_;
  const int t = threadIdx.x;
  T* sM = pool;  // [plane][closed rows of RX columns, outside rows of RC columns]
  T* sL = sM + K * G::SM;
  T* sB = sL + K * G::SC;
  {
    // z pass: column (row, col) of the box; boundary nodes and what lies outside count as 0
    const int z0 = (cz - 2) * K, zlo = max(z0, 0), ps = n1 * n1 * (int)sizeof(Tin);
    const __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<Tin*>(x) + (size_t)zlo * n1 * n1, (short)0, (min(z0 + W, n1) - zlo) * ps, 0x00020000);
    for (int it = t; it < G::NZ; it += NTH) {
      const bool closed_row = it < RC * RX;
      const int ie = it - RC * RX, r = closed_row ? it / RX : ie / RC, col = closed_row ? it - r * RX : ie - r * RC;
      const int gx = (cx0 - 2) * K + col + (closed_row ? 0 : K);
      const int gy = (cy0 - 2) * K + (closed_row ? K + r : r < K ? r : r + RC);
      const unsigned o = gx >= 1 && gx <= n1 - 2 && gy >= 1 && gy <= n1 - 2
                             ? (unsigned)(gy * n1 + gx) * (unsigned)sizeof(Tin)
                             : tile2::kOff;
      T v[W];
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const int gz = z0 + j;
        const bool on = gz >= 1 && gz <= n1 - 2;
        const int so = on ? (gz - zlo) * ps : 0;
        const int oo = on ? (int)o : (int)tile2::kOff;
        if constexpr (sizeof(Tin) == 8)
          v[j] = (T)__builtin_bit_cast(Tin, __builtin_amdgcn_raw_buffer_load_b64(buf, oo, so, 0));
        else
          v[j] = (T)__builtin_bit_cast(Tin, __builtin_amdgcn_raw_buffer_load_b32(buf, oo, so, 0));
      }
      T* m = sM + (closed_row ? r * RXP : RC * RXP + r * RCP) + col;
#pragma unroll
      for (int p = 0; p < K; ++p) m[p * G::SM] = band_ref<T, 0, K>(v + 2 * K + p, p);
      if (closed_row && col >= K && col < K + RC) {
        const int c = r * RCP + col - K;
#pragma unroll
        for (int p = 0; p < K; ++p) sL[p * G::SC + c] = band_ref<T, 1, K>(v + 2 * K + p, p);
        T a[K];
#pragma unroll
        for (int p = 0; p < K; ++p) a[p] = band_ref<T, 2, K>(v + 2 * K + p, p);
        ref::boundary_b<T, K>(a, v + 2 * K, cz, N);
#pragma unroll
        for (int p = 0; p < K; ++p) sB[p * G::SC + c] = a[p];
      }
    }
  }
  __syncthreads();
  // x pass: closed rows (plane, row, cell) from the first thread on, outside rows from the last one down
  T v1[K], v2[K], v3[K], w3[K];
  const int te = NTH - 1 - t;
  const int xp = t / (RC * TC), xr = t % RC, xw = (t / RC) % TC;
  const int ep = te / (E * TC), er = te % E, ew = (te / E) % TC;
  if (t < G::XC) {
    T in[W], l[C];
    const T* m = sM + xp * G::SM + xr * RXP + xw * K;
#pragma unroll
    for (int j = 0; j < W; ++j) in[j] = m[j];
#pragma unroll
    for (int p = 0; p < K; ++p) v3[p] = band_ref<T, 0, K>(in + 2 * K + p, p);
#pragma unroll
    for (int p = 0; p < K; ++p) v2[p] = band_ref<T, 1, K>(in + 2 * K + p, p);
#pragma unroll
    for (int p = 0; p < K; ++p) v1[p] = band_ref<T, 2, K>(in + 2 * K + p, p);
    ref::boundary_b<T, K>(v1, in + 2 * K, cx0 + xw, N);
    m = sL + xp * G::SC + xr * RCP + xw * K;
#pragma unroll
    for (int j = 0; j < C; ++j) l[j] = m[j];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      v2[p] = T(2) * (v2[p] + band_ref<T, 0, K>(l + K + p, p));
      v1[p] += T(2) * band_ref<T, 1, K>(l + K + p, p);
    }
    m = sB + xp * G::SC + xr * RCP + xw * K;
#pragma unroll
    for (int j = 0; j < C; ++j) l[j] = m[j];
#pragma unroll
    for (int p = 0; p < K; ++p) v1[p] += band_ref<T, 0, K>(l + K + p, p);
  }
  if (te < G::XE) {
    T in[C];
    const T* m = sM + ep * G::SM + RC * RXP + er * RCP + ew * K;
#pragma unroll
    for (int j = 0; j < C; ++j) in[j] = m[j];
#pragma unroll
    for (int p = 0; p < K; ++p) w3[p] = band_ref<T, 0, K>(in + K + p, p);
  }
  __syncthreads();  // V goes over the planes just read
  T* sV3 = pool;  // [plane][row of the box][column]
  T* sV1 = sV3 + K * RX * TXP;
  T* sV2 = sV1 + K * RC * TXP;
  if (t < G::XC) {
#pragma unroll
    for (int p = 0; p < K; ++p) {
      sV3[(xp * RX + K + xr) * TXP + xw * K + p] = v3[p];
      sV1[(xp * RC + xr) * TXP + xw * K + p] = v1[p];
      sV2[(xp * RC + xr) * TXP + xw * K + p] = v2[p];
    }
  }
  if (te < G::XE) {
#pragma unroll
    for (int p = 0; p < K; ++p) sV3[(ep * RX + (er < K ? er : er + RC)) * TXP + ew * K + p] = w3[p];
  }
  __syncthreads();
  // y pass: (plane, cell, column), columns fastest across lanes
  for (int it = t; it < G::NY; it += NTH) {
    const int p2 = it / (TX * TC), l = it % TX, w = (it / TX) % TC;
    T a[K], in[W];
    const T* m = sV3 + (p2 * RX + w * K) * TXP + l;
#pragma unroll
    for (int j = 0; j < W; ++j) in[j] = m[j * TXP];
#pragma unroll
    for (int p = 0; p < K; ++p) a[p] = band_ref<T, 2, K>(in + 2 * K + p, p);
    ref::boundary_b<T, K>(a, in + 2 * K, cy0 + w, N);
    m = sV1 + (p2 * RC + w * K) * TXP + l;
#pragma unroll
    for (int j = 0; j < C; ++j) in[j] = m[j * TXP];
#pragma unroll
    for (int p = 0; p < K; ++p) a[p] += band_ref<T, 0, K>(in + K + p, p);
    m = sV2 + (p2 * RC + w * K) * TXP + l;
#pragma unroll
    for (int j = 0; j < C; ++j) in[j] = m[j * TXP];
    const int gx = cx0 * K + l, gz = cz * K + p2;
    const size_t g = ((size_t)gz * n1 + (cy0 + w) * K) * n1 + gx;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const bool inner = gx > 0 && gz > 0 && (p > 0 || cy0 + w > 0);
      const T v = scale * (a[p] + band_ref<T, 1, K>(in + K + p, p));
      y[g + (size_t)p * n1] = inner ? (RES ? b[g + (size_t)p * n1] - v : v) : T(0);
    }
  }
}

template <typename Tin, typename T, int K>
hipError_t apply3d_box_k(int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s) {
  using G = Box<K>;
  const int n1 = K * N + 1, nt = N / G::TC, total = nt * nt * N, grid = total + face_blocks<G::NTH>(n1);
  if (b)
    apply3d_box_kernel<Tin, T, K, G::NTH, true>
        <<<grid, G::NTH, 0, s>>>(x, b, y, N, n1, c.hinv, nt, tile2::magic(nt), total);
  else
    apply3d_box_kernel<Tin, T, K, G::NTH, false>
        <<<grid, G::NTH, 0, s>>>(x, b, y, N, n1, c.hinv, nt, tile2::magic(nt), total);
  return hipGetLastError();
}

}  // namespace

template <typename Tin, typename T>
hipError_t launch_apply3d_box(int k, int N, const LevelCoef<T>& c, const Tin* x, const T* b, T* y, hipStream_t s) {
#define CALL(K) apply3d_box_k<Tin, T, K>(N, c, x, b, y, s)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

template hipError_t launch_apply3d_box<double, double>(int, int, const LevelCoef<double>&, const double*,
                                                       const double*, double*, hipStream_t);
template hipError_t launch_apply3d_box<float, double>(int, int, const LevelCoef<double>&, const float*,
                                                      const double*, double*, hipStream_t);
template hipError_t launch_apply3d_box<float, float>(int, int, const LevelCoef<float>&, const float*, const float*,
                                                     float*, hipStream_t);

}  // namespace c0ip
