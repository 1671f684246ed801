// 3D transfers between nested meshes in one launch each, with the compile-time
// embedding table pt[s][p][a] (value of coarse basis a at the fine node of
// position p in fine cell s of the coarse cell): restriction b_c = P^T r_f and
// prolongation x_f += P e_c.  A workgroup owns TC x TC coarse cells of one
// layer; a z pass per column straight from memory, then an x pass and a y pass
// in LDS.  One launch per axis with both intermediate results in memory took
// 66 us to restrict and 53 to prolong at Q2 128^3 float32, against 27 and 25
// now, and 14 on small meshes, against 5.
#include "faces3d.h"
#include "kernels.h"
#include "tile2d.h"

namespace c0ip {
namespace {

constexpr int kNth = 256;

// Coarse cells per axis of a workgroup's tile, as LDS allows.
template <int K> struct TransferTile { static constexpr int TC = K <= 3 ? 4 : K <= 5 ? 2 : 1; };

template <typename T, int K>
__global__ __launch_bounds__(kNth) void restrict3d_kernel(const T* __restrict__ rf, T* __restrict__ bc, int Nc,
                                                          int nt, unsigned mt, int total) {
  constexpr int TC = TransferTile<K>::TC, S = 2 * K * (TC + 1), SP = S | 1, TX = TC * K, TXP = TX | 1;
  const int nf = 2 * K * Nc + 1, nc = K * Nc + 1;
  if ((int)blockIdx.x >= total) {
    zero_faces<T, kNth>(bc, nc, blockIdx.x - total);
    return;
  }
  __shared__ T sF[K * S * SP];
  __shared__ T sT[K * S * TXP];
  const unsigned q = tile2::xcd_order(blockIdx.x, total), yz = tile2::quotient(q, mt), cz_ = tile2::quotient(yz, mt);
  const int cx0 = (int)(q - yz * nt) * TC, cy0 = (int)(yz - cz_ * nt) * TC, cz = (int)cz_;
  const size_t pl = (size_t)nf * nf;
  for (int it = threadIdx.x; it < S * S; it += kNth) {
    const int j = it / S, i = it - j * S;
    const int gx = 2 * K * (cx0 - 1) + i, gy = 2 * K * (cy0 - 1) + j;
    const bool on = gx >= 0 && gx < nf && gy >= 0 && gy < nf;
    const T* p = rf + ((size_t)(2 * K * cz) * nf + (on ? gy : 0)) * nf + (on ? gx : 0);
    T in[4 * K], o[K];
#pragma unroll
    for (int z = 0; z < 4 * K; ++z) in[z] = z >= 2 * K || cz > 0 ? p[(int64_t)(z - 2 * K) * (int64_t)pl] : T(0);
    tile2::gather<T, K>(in, o);
#pragma unroll
    for (int a = 0; a < K; ++a) sF[(a * S + j) * SP + i] = on ? o[a] : T(0);
  }
  __syncthreads();
  for (int it = threadIdx.x; it < K * S * TC; it += kNth) {
    const int row = it % (K * S), c = it / (K * S);
    T in[4 * K], o[K];
#pragma unroll
    for (int i = 0; i < 4 * K; ++i) in[i] = sF[row * SP + 2 * K * c + i];
    tile2::gather<T, K>(in, o);
#pragma unroll
    for (int a = 0; a < K; ++a) sT[row * TXP + c * K + a] = o[a];
  }
  __syncthreads();
  for (int it = threadIdx.x; it < K * TC * TX; it += kNth) {
    const int l = it % TX, c = (it / TX) % TC, a0 = it / (TX * TC);
    const int gx = cx0 * K + l, gy = (cy0 + c) * K, gz = cz * K + a0;
    if (cx0 * K + l >= nc - 1 || cy0 + c >= Nc) continue;
    T in[4 * K], o[K];
#pragma unroll
    for (int i = 0; i < 4 * K; ++i) in[i] = sT[(a0 * S + 2 * K * c + i) * TXP + l];
    tile2::gather<T, K>(in, o);
#pragma unroll
    for (int a = 0; a < K; ++a)
      bc[((size_t)gz * nc + gy + a) * nc + gx] = gx > 0 && gy + a > 0 && gz > 0 ? o[a] : T(0);
  }
}

template <typename T, int K>
__global__ __launch_bounds__(kNth) void prolong3d_kernel(const T* __restrict__ ec, T* __restrict__ xf, int Nc, int nt,
                                                         unsigned mt) {
  constexpr int TC = TransferTile<K>::TC, CW = TC * K + 1, CP = CW | 1, FT = 2 * K * TC, FP = FT | 1;
  const int nf = 2 * K * Nc + 1, nc = K * Nc + 1;
  __shared__ T sC[2 * K * CW * CP];
  __shared__ T sT[2 * K * CW * FP];
  const unsigned q = tile2::xcd_order(blockIdx.x, gridDim.x), yz = tile2::quotient(q, mt),
                 cz_ = tile2::quotient(yz, mt);
  const int cx0 = (int)(q - yz * nt) * TC, cy0 = (int)(yz - cz_ * nt) * TC, cz = (int)cz_;
  const size_t pl = (size_t)nc * nc;
  for (int it = threadIdx.x; it < CW * CW; it += kNth) {
    const int j = it / CW, i = it - j * CW, gx = cx0 * K + i, gy = cy0 * K + j;
    const bool on = gx < nc && gy < nc;
    const T* p = ec + ((size_t)(K * cz) * nc + (on ? gy : 0)) * nc + (on ? gx : 0);
    T in[K + 1], o[2 * K];
#pragma unroll
    for (int a = 0; a <= K; ++a) in[a] = p[a * pl];
    tile2::spread<T, K>(in, o);
#pragma unroll
    for (int z = 0; z < 2 * K; ++z) sC[(z * CW + j) * CP + i] = on ? o[z] : T(0);
  }
  __syncthreads();
  for (int it = threadIdx.x; it < 2 * K * CW * TC; it += kNth) {
    const int row = it % (2 * K * CW), c = it / (2 * K * CW);
    T in[K + 1], o[2 * K];
#pragma unroll
    for (int a = 0; a <= K; ++a) in[a] = sC[row * CP + c * K + a];
    tile2::spread<T, K>(in, o);
#pragma unroll
    for (int i = 0; i < 2 * K; ++i) sT[row * FP + 2 * K * c + i] = o[i];
  }
  __syncthreads();
  for (int it = threadIdx.x; it < 2 * K * TC * FT; it += kNth) {
    const int l = it % FT, c = (it / FT) % TC, z = it / (FT * TC);
    const int gx = 2 * K * cx0 + l, gy = 2 * K * (cy0 + c), gz = 2 * K * cz + z;
    if (gx == 0 || gx >= nf - 1 || cy0 + c >= Nc || gz == 0) continue;
    T in[K + 1], o[2 * K];
#pragma unroll
    for (int a = 0; a <= K; ++a) in[a] = sT[(z * CW + c * K + a) * FP + l];
    tile2::spread<T, K>(in, o);
    T* x = xf + ((size_t)gz * nf + gy) * nf + gx;
    T v[2 * K];
#pragma unroll
    for (int i = 0; i < 2 * K; ++i) v[i] = x[(size_t)i * nf];
#pragma unroll
    for (int i = 0; i < 2 * K; ++i)
      if (i > 0 || gy > 0) x[(size_t)i * nf] = v[i] + o[i];
  }
}

template <typename T, int K>
hipError_t restrict3d_k(int Nc, const T* rf, T* bc, hipStream_t s) {
  constexpr int TC = TransferTile<K>::TC;
  const int nt = (Nc + TC - 1) / TC, total = nt * nt * Nc;
  restrict3d_kernel<T, K><<<total + face_blocks<kNth>(K * Nc + 1), kNth, 0, s>>>(rf, bc, Nc, nt, tile2::magic(nt),
                                                                                total);
  return hipGetLastError();
}
template <typename T, int K>
hipError_t prolong3d_k(int Nc, const T* ec, T* xf, hipStream_t s) {
  constexpr int TC = TransferTile<K>::TC;
  const int nt = (Nc + TC - 1) / TC;
  prolong3d_kernel<T, K><<<nt * nt * Nc, kNth, 0, s>>>(ec, xf, Nc, nt, tile2::magic(nt));
  return hipGetLastError();
}

// fine vectors of 2^31 entries and more are refused
bool fits(int k, int Nc) {
  const int64_t nf = (int64_t)k * 2 * Nc + 1;
  return nf * nf * nf < (1ll << 31);
}

}  // namespace

template <typename T>
hipError_t launch_restrict3d(int k, int Nc, const T* rf, T* bc, hipStream_t s) {
  if (!fits(k, Nc)) return hipErrorInvalidValue;
#define CALL(K) restrict3d_k<T, K>(Nc, rf, bc, s)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}
template <typename T>
hipError_t launch_prolong3d(int k, int Nc, const T* ec, T* xf, hipStream_t s) {
  if (!fits(k, Nc)) return hipErrorInvalidValue;
#define CALL(K) prolong3d_k<T, K>(Nc, ec, xf, s)
  C0IP_DISPATCH_K(k, CALL)
#undef CALL
}

template hipError_t launch_restrict3d<double>(int, int, const double*, double*, hipStream_t);
template hipError_t launch_restrict3d<float>(int, int, const float*, float*, hipStream_t);
template hipError_t launch_prolong3d<double>(int, int, const double*, double*, hipStream_t);
template hipError_t launch_prolong3d<float>(int, int, const float*, float*, hipStream_t);

}  // namespace c0ip
