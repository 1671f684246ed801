// The lowest levels of the V-cycle (Algorithm 1) in one workgroup per system
// for the default penalty, with every vector of those levels in LDS.
//
// Below a few thousand DoFs per level each kernel of the V-cycle is bound by
// its own launch and memory latency (about 5 us each, three per level).  Here
// levels 0..LT run in a single launch: the right-hand side of level LT is
// read once, pre-smoothing, residual, restriction, the coarse solve,
// prolongation and post-smoothing of every level below run from LDS with
// workgroup barriers between phases, and x of level LT is written once.  The
// phases are those of tile2d.h with the whole level as the tile: two for the
// operator, three for the patch solves, two for a transfer.
//
// Work split: a wave owns a cell (or vertex, or coarse cell) along one axis
// and its lanes run along the other, so cell positions, boundary rows, patch
// variants and the eigenbasis are wave-uniform, coefficients compile-time,
// and no index needs a division.  x is kept with 2k zero columns on each
// side; T's halo rows are zeroed with each x pass.
#include "kernels.h"
#include "tile2d.h"

namespace c0ip {
namespace {

using ref::band_ref;
using ref::mad;
using tile::Band;
using tile::variant;

// Threads of the workgroup: 1024 leave 128 registers each, which float64
// overruns from k = 3 on.  At k = 3 the waves are worth more (Q3 16^2 V-cycle
// 61.2 us against 64.3, 2+2 steps 109 against 115), at k = 4 they are not.
template <typename T, int K>
constexpr int kThreadsOf = sizeof(T) == 8 && K >= 4 ? 512 : 1024;

// LDS layout in T elements; the same function sizes the launch.
struct RefLayout {
  int x[kTailMaxLevels], b[kTailMaxLevels], q[kTailMaxLevels], lam[kTailMaxLevels];
  int r, s;  // residual; scratch: the operator's x passes, the patch modes, or a transfer's x pass
  int a0;    // the float64 level-0 inverse, in doubles
  int bytes;
};

inline int imax(int a, int b) { return a > b ? a : b; }

inline RefLayout ref_layout(int k, int LT, int tsize) {
  RefLayout L{};
  const int n = 2 * k - 1;
  int off = 0, scr = 0;
  for (int l = 0; l <= LT; ++l) {
    const int N = 2 << l, n1 = k * N + 1, xp = (N - 1) * n;  // xp is odd
    L.x[l] = off;
    off += n1 * (n1 + 4 * k);
    L.b[l] = off;
    off += n1 * n1;
    L.q[l] = off;
    off += 4 * n * n;
    L.lam[l] = off;
    off += 4 * n;
    scr = imax(scr, (n1 + 4 * k) * n1 + 2 * (n1 + 2 * k) * n1);
    scr = imax(scr, (n1 - 2) * xp + (N - 1) * n * xp);
  }
  const int n1 = k * (2 << LT) + 1;
  L.r = off;
  off += n1 * n1;
  L.s = off;
  off += scr;
  const int tbytes = (off * tsize + 15) / 16 * 16;
  L.a0 = tbytes / 8;
  L.bytes = tbytes + n * n * n * n * 8;
  return L;
}

template <typename T, int K>
struct Tail {
  static constexpr int n = 2 * K - 1, NN = n * n, kTailThreads = kThreadsOf<T, K>, kWaves = kTailThreads / 64;
  static __device__ __forceinline__ int wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
  static __device__ __forceinline__ int lane() { return threadIdx.x & 63; }

  // T = X M_x, X L_x, X B_x of every row; halo rows of T are 0.
  static __device__ __forceinline__ void op_x(int N, const T* x, T* s) {
    const int n1 = K * N + 1, SX = n1 + 4 * K;
    T* sM = s + 2 * K * n1;
    T* sL = s + (n1 + 4 * K) * n1 + K * n1;
    T* sB = sL + (n1 + 2 * K) * n1;
    for (int e = threadIdx.x; e < 2 * K * n1; e += kTailThreads) {
      s[e] = T(0);
      sM[n1 * n1 + e] = T(0);
      if (e < K * n1) sL[e - K * n1] = sL[n1 * n1 + e] = sB[e - K * n1] = sB[n1 * n1 + e] = T(0);
    }
    for (int c = wave(); c < N; c += kWaves)
      for (int r = lane(); r < n1; r += 64) {
        T in[4 * K + K];
#pragma unroll
        for (int j = 0; j < 5 * K; ++j) in[j] = x[r * SX + c * K + j];
        const T* v = in + 2 * K;
        T a[K];
        const int o = r * n1 + c * K;
#pragma unroll
        for (int p = 0; p < K; ++p) {
          sM[o + p] = band_ref<T, 0, K>(v + p, p);
          sL[o + p] = band_ref<T, 1, K>(v + p, p);
          a[p] = band_ref<T, 2, K>(v + p, p);
        }
        ref::boundary_b<T, K>(a, v, c, N);
#pragma unroll
        for (int p = 0; p < K; ++p) sB[o + p] = a[p];
      }
    // nothing reads the last column (boundary node)
  }

  // r = b - A x on the interior nodes (0 on the boundary).
  static __device__ __forceinline__ void op_y(int N, const T* s, const T* b, T* r, T scale) {
    const int n1 = K * N + 1, NK = n1 - 1;
    const T* sM = s + 2 * K * n1;
    const T* sL = s + (n1 + 4 * K) * n1 + K * n1;
    const T* sB = sL + (n1 + 2 * K) * n1;
    for (int c = wave(); c < N; c += kWaves)
      for (int l = lane(); l < NK; l += 64) {
        T acc[K];
        {
          T t[3 * K];
#pragma unroll
          for (int j = 0; j < 3 * K; ++j) t[j] = sB[((c - 1) * K + j) * n1 + l];
#pragma unroll
          for (int p = 0; p < K; ++p) acc[p] = band_ref<T, 0, K>(t + p + K, p);
        }
        {
          T t[3 * K];
#pragma unroll
          for (int j = 0; j < 3 * K; ++j) t[j] = sL[((c - 1) * K + j) * n1 + l];
#pragma unroll
          for (int p = 0; p < K; ++p) acc[p] += T(2) * band_ref<T, 1, K>(t + p + K, p);
        }
        {
          T t[5 * K], a[K];
#pragma unroll
          for (int j = 0; j < 5 * K; ++j) t[j] = sM[((c - 2) * K + j) * n1 + l];
#pragma unroll
          for (int p = 0; p < K; ++p) a[p] = band_ref<T, 2, K>(t + p + 2 * K, p);
          ref::boundary_b<T, K>(a, t + 2 * K, c, N);
#pragma unroll
          for (int p = 0; p < K; ++p) acc[p] += a[p];
        }
#pragma unroll
        for (int p = 0; p < K; ++p) {
          const int o = (c * K + p) * n1 + l;
          r[o] = l >= 1 && c * K + p >= 1 ? b[o] - scale * acc[p] : T(0);
        }
      }
  }

  // Patch solves from r (row stride n1): x modes, then y solves.
  static __device__ __forceinline__ void fd_x(int N, const T* r, T* s, const T* Q) {
    const int n1 = K * N + 1, XP = (N - 1) * n;
    for (int v = 1 + wave(); v < N; v += kWaves) {
      const T* q = Q + variant(v, N) * NN;
      for (int row = lane(); row < n1 - 2; row += 64) {
        T in[n], out[n];
#pragma unroll
        for (int a = 0; a < n; ++a) in[a] = r[(row + 1) * n1 + (v - 1) * K + 1 + a];
        tile2::tr1<T, n, true>(q, in, out);
#pragma unroll
        for (int a = 0; a < n; ++a) s[row * XP + (v - 1) * n + a] = out[a];
      }
    }
  }
  static __device__ __forceinline__ void fd_y(int N, T* s, const T* Q, const T* lam) {
    const int n1 = K * N + 1, XP = (N - 1) * n;
    T* sU = s + (n1 - 2) * XP;
    for (int v = 1 + wave(); v < N; v += kWaves) {
      const int ty = variant(v, N);
      const T* q = Q + ty * NN;
      for (int col = lane(); col < XP; col += 64) {
        const int px = col / n, mx = col - px * n;
        const T lx = lam[variant(px + 1, N) * n + mx];
        T in[n], w[n];
#pragma unroll
        for (int a = 0; a < n; ++a) in[a] = s[((v - 1) * K + a) * XP + col];
        tile2::tr1<T, n, true>(q, in, w);
#pragma unroll
        for (int m = 0; m < n; ++m) w[m] /= lx + lam[ty * n + m];
        tile2::tr1<T, n, false>(q, w, in);
#pragma unroll
        for (int a = 0; a < n; ++a) sU[((v - 1) * n + a) * XP + col] = in[a];
      }
    }
  }
  // x = (zero ? 0 : x) + omega * corrections on the interior nodes.
  static __device__ __forceinline__ void fd_out(int N, const T* s, const T* Q, T* x, T omega, bool zero) {
    const int n1 = K * N + 1, XP = (N - 1) * n, SX = n1 + 4 * K, NK = n1 - 1;
    const T* sU = s + (n1 - 2) * XP;
    for (int c = wave(); c < N; c += kWaves) {
      // patch columns of vertices c and c + 1 (absent at the boundary)
      const bool ha = c >= 1, hb = c + 1 <= N - 1;
      const T* qa = Q + (ha ? variant(c, N) : 0) * NN;
      const T* qb = Q + (hb ? variant(c + 1, N) : 0) * NN;
      for (int gy = 1 + lane(); gy < NK; gy += 64) {
        const int my = gy / K, ry = gy - my * K;
        const T* ua = sU + ((my - 1) * n + K - 1 + ry) * XP;  // vertex row my
        const T* ub = sU + (my * n + ry - 1) * XP;            // vertex row my + 1
        const bool va = my >= 1, vb = ry > 0 && my + 1 <= N - 1;
        T wa[n], wb[n];
#pragma unroll
        for (int m = 0; m < n; ++m) {
          wa[m] = ha && va ? ua[(c - 1) * n + m] : T(0);
          wb[m] = hb && va ? ua[c * n + m] : T(0);
        }
        if (vb) {
#pragma unroll
          for (int m = 0; m < n; ++m) {
            if (ha) wa[m] += ub[(c - 1) * n + m];
            if (hb) wb[m] += ub[c * n + m];
          }
        }
        T* xo = x + gy * SX + 2 * K + c * K;
#pragma unroll
        for (int p = 0; p < K; ++p) {
          T a = qa[(K - 1 + p) * n] * wa[0];
#pragma unroll
          for (int m = 1; m < n; ++m) a = mad(qa[(K - 1 + p) * n + m], wa[m], a);
          if (p > 0) {
#pragma unroll
            for (int m = 0; m < n; ++m) a = mad(qb[(p > 0 ? p - 1 : 0) * n + m], wb[m], a);
          }
          if (p > 0 || c > 0) xo[p] = (zero ? T(0) : xo[p]) + omega * a;
        }
      }
    }
  }

  // bc = P^T rf on the coarse interior: S[fine row][coarse column], then along y.
  static __device__ __forceinline__ void restrict_x(int Nc, const T* rf, T* s) {
    const int nf = 2 * K * Nc + 1, nc = K * Nc + 1;
    for (int c = wave(); c < Nc; c += kWaves)
      for (int row = lane(); row < nf - 1; row += 64) {
        T in[4 * K];  // the coarse cell to the left and this one
#pragma unroll
        for (int q = 0; q < 4 * K; ++q) in[q] = q >= 2 * K || c > 0 ? rf[row * nf + 2 * (c - 1) * K + q] : T(0);
#pragma unroll
        for (int a = 0; a < K; ++a) s[row * nc + c * K + a] = gather(in, a);
      }
  }
  static __device__ __forceinline__ void restrict_y(int Nc, const T* s, T* bc) {
    const int nc = K * Nc + 1;
    for (int c = wave(); c < Nc; c += kWaves)
      for (int col = lane(); col < nc; col += 64) {
        T in[4 * K];
#pragma unroll
        for (int q = 0; q < 4 * K; ++q)
          in[q] = col < nc - 1 && (q >= 2 * K || c > 0) ? s[(2 * (c - 1) * K + q) * nc + col] : T(0);
#pragma unroll
        for (int a = 0; a < K; ++a) bc[(c * K + a) * nc + col] = col >= 1 && c * K + a >= 1 ? gather(in, a) : T(0);
      }
  }
  static __device__ __forceinline__ T gather(const T (&in)[4 * K], int a) {
    T v = (T)RefCoef<K>::pt[0][0][a] * in[2 * K];
#pragma unroll
    for (int q = 1; q < 2 * K; ++q) v = mad((T)RefCoef<K>::pt[q / K][q % K][a], in[2 * K + q], v);
    if (a == 0) {
#pragma unroll
      for (int q = 0; q < 2 * K; ++q) v = mad((T)RefCoef<K>::pt[q / K][q % K][K], in[q], v);
    }
    return v;
  }
  // x += P ec: S[coarse row][fine column], then along y.
  static __device__ __forceinline__ void prolong_x(int Nc, const T* ec, T* s) {
    const int nf = 2 * K * Nc + 1, nc = K * Nc + 1, SC = nc + 4 * K;
    for (int c = wave(); c < Nc; c += kWaves)
      for (int row = lane(); row < nc; row += 64) {
        T in[K + 1];
#pragma unroll
        for (int a = 0; a <= K; ++a) in[a] = ec[row * SC + 2 * K + c * K + a];
#pragma unroll
        for (int q = 0; q < 2 * K; ++q) s[row * nf + 2 * c * K + q] = spread(in, q);
      }
  }
  static __device__ __forceinline__ void prolong_y(int Nc, const T* s, T* x) {
    const int nf = 2 * K * Nc + 1, SX = nf + 4 * K;
    for (int c = wave(); c < Nc; c += kWaves)
      for (int col = 1 + lane(); col < nf - 1; col += 64) {
        T in[K + 1];
#pragma unroll
        for (int a = 0; a <= K; ++a) in[a] = s[(c * K + a) * nf + col];
#pragma unroll
        for (int q = 0; q < 2 * K; ++q)
          if (q > 0 || c > 0) x[(2 * c * K + q) * SX + 2 * K + col] += spread(in, q);
      }
  }
  static __device__ __forceinline__ T spread(const T (&in)[K + 1], int q) {
    T v = (T)RefCoef<K>::pt[q / K][q % K][0] * in[0];
#pragma unroll
    for (int a = 1; a <= K; ++a) v = mad((T)RefCoef<K>::pt[q / K][q % K][a], in[a], v);
    return v;
  }
};

// Bound by the instruction latency of a single compute unit's waves (about 40
// phases of 1000 to 4500 cycles).  Q3 levels 16^2 .. 2^2 float32 55 -> 43 us,
// Q4 118 -> 53, Q2 32^2 .. 2^2 69 -> 51, Q4 8^2 .. 2^2 float64 59 -> 45; Q3
// 16^2 float64 65 -> 64.  L comes as an argument: its per-level entries are then scalar loads
// (computed here, the arrays would live in scratch memory).
template <typename T, int K, int NTH>
__global__ __launch_bounds__(NTH) void vtail_ref_kernel(TailParams<T> P, TailIO<T> io, RefLayout L) {
  using L_ = Tail<T, K>;
  constexpr int kTailThreads = L_::kTailThreads, kWaves = L_::kWaves;
  extern __shared__ __align__(16) unsigned char smem[];
  const int sys = blockIdx.x;
  if (io.active && !io.active[sys]) return;
  int top = 0;
  for (int l = 1; l <= P.LT; ++l)
    if (sys < io.nA[l]) top = l;
  T* S = reinterpret_cast<T*>(smem);
  double* A0 = reinterpret_cast<double*>(smem) + L.a0;
  constexpr int n = 2 * K - 1, n0 = n * n;
  const int n1t = K * (2 << top) + 1;
  {
    // eigendata, coarse inverse and right-hand side: every load of a group is issued before its stores
    constexpr int NA = (n0 * n0 + kTailThreads - 1) / kTailThreads;
    const int t = threadIdx.x;
    T q[kTailMaxLevels], lam[kTailMaxLevels];
    double a0[NA];
#pragma unroll
    for (int l = 0; l < kTailMaxLevels; ++l) {
      q[l] = l <= top && t < 4 * n0 ? P.Q[l][t] : T(0);
      lam[l] = l <= top && t < 4 * n ? P.lam[l][t] : T(0);
    }
#pragma unroll
    for (int u = 0; u < NA; ++u)
      a0[u] = P.coarse_mode == 0 && t + u * kTailThreads < n0 * n0 ? P.Ainv[t + u * kTailThreads] : 0.0;
    const T* src = io.b[top] + (int64_t)sys * io.stride[top];
    T* dst = S + L.b[top];
    for (int e0 = t; e0 < n1t * n1t; e0 += 4 * kTailThreads) {
      T v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = e0 + u * kTailThreads < n1t * n1t ? src[e0 + u * kTailThreads] : T(0);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (e0 + u * kTailThreads < n1t * n1t) dst[e0 + u * kTailThreads] = v[u];
    }
#pragma unroll
    for (int l = 0; l < kTailMaxLevels; ++l) {
      if (l <= top && t < 4 * n0) S[L.q[l] + t] = q[l];
      if (l <= top && t < 4 * n) S[L.lam[l] + t] = lam[l];
    }
#pragma unroll
    for (int u = 0; u < NA; ++u)
      if (t + u * kTailThreads < n0 * n0) A0[t + u * kTailThreads] = a0[u];
    for (int l = 0; l <= top; ++l) {
      const int n1 = K * (2 << l) + 1;
      for (int e = t; e < n1 * (n1 + 4 * K); e += kTailThreads) S[L.x[l] + e] = T(0);
    }
  }
  __syncthreads();
  T* r = S + L.r;
  T* s = S + L.s;
  // The V-cycle as one loop over groups of phases, so that the code of each
  // phase is there once: what a workgroup waits for on these levels is mostly
  // instructions that are not in the cache yet, and every level runs the same.
  //   going down: pre groups [residual unless the first, solves], then
  //     [residual, restriction]; the coarse solve below level 1;
  //   going up: post groups [prolongation if the first, residual, solves]
  //     ([prolongation] alone for post = 0).
  int l = top, st = 0;
  bool up = false;
  while (l <= top) {
    const bool coarse = l == 0;
    const bool pro = up && st == 0, sol = coarse ? P.coarse_mode != 0 : (up ? P.post > 0 : st < P.pre);
    const bool res = !coarse && (up ? P.post > 0 : st > 0 || !sol), rst = !coarse && !up && !sol;
    const bool zero = !up && st == 0;
    const int N = 2 << l, Nh = 1 << l;
    T* x = S + L.x[l];
    const T* Q = S + L.q[l];
    if (pro) {
      L_::prolong_x(Nh, S + L.x[l - 1], s);
      __syncthreads();
      L_::prolong_y(Nh, s, x);
      __syncthreads();
    }
    if (res) {
      L_::op_x(N, x, s);
      __syncthreads();
      L_::op_y(N, s, S + L.b[l], r, T(N) * T(N));  // 1 / h^2
      __syncthreads();
    }
    if (sol) {
      L_::fd_x(N, zero ? S + L.b[l] : r, s, Q);
      __syncthreads();
      L_::fd_y(N, s, Q, S + L.lam[l]);
      __syncthreads();
      L_::fd_out(N, s, Q, x, coarse ? T(1) : P.omega, zero);
      __syncthreads();
    }
    if (rst) {
      L_::restrict_x(Nh, r, s);
      __syncthreads();
      L_::restrict_y(Nh, s, S + L.b[l - 1]);
      __syncthreads();
    }
    if (coarse && !sol) {
      const T* b0 = S + L.b[0];
      constexpr int n1 = 2 * K + 1;
      for (int u = threadIdx.x; u < n0; u += kTailThreads) {
        double a = 0;
#pragma unroll
        for (int c = 0; c < n0; ++c) a += A0[u * n0 + c] * (double)b0[(c / n + 1) * n1 + c % n + 1];
        S[L.x[0] + (u / n + 1) * (n1 + 4 * K) + 2 * K + u % n + 1] = (T)a;
      }
      __syncthreads();
    }
    // the next group
    if (coarse) {
      up = true;
      l = 1;
      st = 0;
    } else if (!up) {
      if (rst) {
        --l;
        st = 0;
      } else {
        ++st;
      }
    } else if (++st >= P.post) {
      ++l;
      st = 0;
    }
  }
  T* out = io.x[top] + (int64_t)sys * io.stride[top];
  for (int j = L_::wave(); j < n1t; j += kWaves)
    for (int i = L_::lane(); i < n1t; i += 64) out[j * n1t + i] = S[L.x[top] + j * (n1t + 4 * K) + 2 * K + i];
}

template <typename T, int K>
hipError_t vtail_ref_k(const TailParams<T>& P, const TailIO<T>& io, int nsys, hipStream_t s) {
  const RefLayout L = ref_layout(K, P.LT, sizeof(T));
  vtail_ref_kernel<T, K, Tail<T, K>::kTailThreads><<<nsys, Tail<T, K>::kTailThreads, L.bytes, s>>>(P, io, L);
  return hipGetLastError();
}

template <typename T, int K>
hipError_t configure_k(int bytes) {
  return hipFuncSetAttribute((const void*)vtail_ref_kernel<T, K, Tail<T, K>::kTailThreads>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

}  // namespace

int tail_ref_bytes(int k, int LT, int elem_size) { return ref_layout(k, LT, elem_size).bytes; }

template <typename T>
hipError_t configure_vtail_ref(int k, int bytes) {
  switch (k) {
    case 2: return configure_k<T, 2>(bytes);
    case 3: return configure_k<T, 3>(bytes);
    case 4: return configure_k<T, 4>(bytes);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_vtail_ref(int k, const TailParams<T>& P, const TailIO<T>& io, int nsys, hipStream_t s) {
  switch (k) {
    case 2: return vtail_ref_k<T, 2>(P, io, nsys, s);
    case 3: return vtail_ref_k<T, 3>(P, io, nsys, s);
    case 4: return vtail_ref_k<T, 4>(P, io, nsys, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t configure_vtail_ref<double>(int, int);
template hipError_t configure_vtail_ref<float>(int, int);
template hipError_t launch_vtail_ref<double>(int, const TailParams<double>&, const TailIO<double>&, int,
                                             hipStream_t);
template hipError_t launch_vtail_ref<float>(int, const TailParams<float>&, const TailIO<float>&, int, hipStream_t);

}  // namespace c0ip
