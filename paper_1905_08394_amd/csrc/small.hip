// Row sweep of small networks: one workgroup contracts a whole row of the
// lattice for one node (or one v value of a node), its running tensor in LDS
// from the first site to the last.
//
// Where a row's tensors hold a few thousand elements, a launch per site spends
// 10 to 20 us on well under a microsecond of work, most of it padding of 128 x
// 128 tiles.  Here a level of the sweep is one launch, which also rescales the
// boundary, or two where the v values of a node are spread over workgroups (the
// second sums over them and rescales).  Site j reads its A operand from one LDS
// buffer and writes C into the other in the layout the next site reads
// (plan.cpp); W comes from L2 as a plain complex matrix, 16 k ahead of the
// products.  These are v_mfma_f32_16x16x4f32 (or f64), four real products per
// complex one, so blocks of 16 waste little on bonds of 2 to 16.  The loops stay
// rolled and the product has three forms only: a row is run once per launch, so
// its instructions are fetched cold.
//
// Bound: at bonds of 8 the matrix units (a row of 4x5 (1+24+1), 512 workgroups,
// two per CU: 19 us of FP32 products in 34 us), below that the chain of dependent
// loads of a row, 8 us.  Kernel time of a call, before -> now: 3x3 (1+8+1) 512
// bitstrings 108 -> 24 us, 4x5 (1+24+1) 64 bitstrings 340 -> 198 us, 48 circuits
// of up to 20 qubits in one group 1000 -> 340 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>

#include "psim_internal.hpp"

namespace psim {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

namespace {

template <typename T>
struct Cx;
template <>
struct Cx<float> {
  typedef f32x2 c;
  typedef f32x4 acc;
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};
template <>
struct Cx<double> {
  typedef f64x2 c;
  typedef f64x4 acc;
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
};

constexpr int kThreads = 256;

// Largest |component| of f[0 .. n) over the workgroup, as an exponent (0 for
// all zeros); every thread gets it.
template <typename T>
__device__ __forceinline__ int max_exponent(const T* f, int n, T* red) {
  T m = 0;
  for (int x = threadIdx.x; x < n; x += blockDim.x) m = fmax(m, fabs(f[x]));
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, red[w]);
  int e = 0;
  if (m > 0) frexp(m, &e);
  return e;
}

// The boundary of a node, f = [d_0 ..][d_{L-1}] in LDS: rescaled by the exact
// power of two that takes its largest component into [1/2, 1), stored as
// [d_{L-1}][d_0 ..], and the node's exponent.
template <typename T>
__device__ __forceinline__ void small_store(const SmallRow& p, int node, const typename Cx<T>::c* f) {
  __shared__ T red[16];
  const int e = max_exponent((const T*)f, 2 * p.F, red);
  const int N = p.site[p.L - 1].dd, M = p.F / N;
  typename Cx<T>::c* F = (typename Cx<T>::c*)p.F_out + (long long)node * p.F;
  for (int x = threadIdx.x; x < p.F; x += blockDim.x) {
    const int n = x / M, m = x - n * M;
    const typename Cx<T>::c c = f[m * N + n];
    F[x] = typename Cx<T>::c{(T)ldexp(c[0], -e), (T)ldexp(c[1], -e)};
  }
  if (threadIdx.x == 0) p.exp_cur[node] = p.exp_prev[p.parent[node]] + e;
}

// The product of one site over the workgroup,
//   C[z][m][n] = sum_k A[z][k1][m][k2] W[k][n]   (rows of C: z, m),
// A and C in LDS, in tiles of TM x TN blocks of 16 x 16 per wave.  Chunks of 16
// k: W comes from global memory one chunk ahead (wnext holds the first chunk of
// this wave's first tile on entry), A from LDS one chunk ahead.  SPLIT: the
// products of a chunk are summed apart first.
template <typename T>
struct Product {
  const typename Cx<T>::c* A;
  const typename Cx<T>::c* W;
  typename Cx<T>::c* C;
  int rows, M, K1, K2, K, N;
};

template <typename T>
struct Chunk {
  typename Cx<T>::c w[4][2];
};

template <typename T, int TN>
__device__ __forceinline__ Chunk<T> load_w(const typename Cx<T>::c* __restrict__ W, int N, int K, int n0, int k0) {
  const int lane = threadIdx.x & 63;
  Chunk<T> c;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = min(n0 + 16 * j + (lane & 15), N - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + 4 * q + (lane >> 4);
      c.w[q][j] = j < TN && k < K ? W[k * N + n] : typename Cx<T>::c{0, 0};
    }
  }
  return c;
}

template <typename T, int TM, int TN, bool SPLIT>
__device__ __forceinline__ void tiles(const Product<T>& p, Chunk<T> wnext) {
  typedef typename Cx<T>::c C;
  typedef typename Cx<T>::acc Acc;
  constexpr int NW = kThreads / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kl = lane >> 4, col = lane & 15;
  const int MK2 = p.M * p.K2;
  const int tn = (p.N + 16 * TN - 1) / (16 * TN), count = (p.rows + 16 * TM - 1) / (16 * TM) * tn;
  const int q4 = 4 / p.K2, step = q4 * MK2 + 4 - q4 * p.K2, r4 = 4 - q4 * p.K2;
  const int kl1 = kl / p.K2, kl2 = kl - kl1 * p.K2;
  for (int t = wave; t < count; t += NW) {
    const int mt = t / tn, nt = t - mt * tn;
    int am[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = min(16 * (mt * TM + i) + col, p.rows - 1), z = row / p.M;
      am[i] = (z * p.K1 * p.M + row - z * p.M) * p.K2;
    }
    int k2 = kl2, at = kl1 * MK2 + kl2, ka = kl;
    C a[4][TM], anext[4][TM], w[4][TN];
    auto load_a = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int i = 0; i < TM; ++i) anext[q][i] = ka < p.K ? p.A[at + am[i]] : C{0, 0};
        ka += 4;
        k2 += r4;
        at += step;
        if (k2 >= p.K2) {
          k2 -= p.K2;
          at += MK2 - p.K2;
        }
      }
    };
    load_a();
    Acc acc[TM][TN][2];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j][0] = acc[i][j][1] = Acc{0, 0, 0, 0};
    for (int k0 = 0; k0 < p.K; k0 += 16) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[q][i] = anext[q][i];
#pragma unroll
        for (int j = 0; j < TN; ++j) w[q][j] = wnext.w[q][j];
      }
      if (k0 + 16 < p.K) {
        wnext = load_w<T, TN>(p.W, p.N, p.K, 16 * TN * nt, k0 + 16);
        load_a();
      } else if (t + NW < count && (tn > 1 || p.K > 16)) {  // else the next tile's W is this one
        wnext = load_w<T, TN>(p.W, p.N, p.K, 16 * TN * ((t + NW) % tn), 0);
      }
      Acc part[SPLIT ? TM : 1][SPLIT ? TN : 1][2];
      auto& dst = [&]() -> auto& {
        if constexpr (SPLIT) return part;
        else return acc;
      }();
      if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) part[i][j][0] = part[i][j][1] = Acc{0, 0, 0, 0};
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (k0 + 4 * q >= p.K) break;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {  // h = 0: Re a times w, 1: Im a times i w
              dst[i][j][0] = Cx<T>::mma(h ? -a[q][i][1] : a[q][i][0], w[q][j][h], dst[i][j][0]);
              dst[i][j][1] = Cx<T>::mma(a[q][i][h], w[q][j][1 - h], dst[i][j][1]);
            }
      }
      if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            acc[i][j][0] += part[i][j][0];
            acc[i][j][1] += part[i][j][1];
          }
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * (mt * TM + i) + Cx<T>::row(lane, r), n = 16 * (nt * TN + j) + col;
          if (row < p.rows && n < p.N) p.C[row * p.N + n] = C{acc[i][j][0][r], acc[i][j][1][r]};
        }
  }
}

// One row for node g, or for v values [vc * (g % parts), ..) of it where the
// node is spread over Dv / vc workgroups.  All v of the workgroup are rows of
// the same products; the last site sums over them.
template <typename T, bool SPLIT>
__device__ __forceinline__ void small_row_body(const SmallRow& p, int g, typename Cx<T>::c* lds) {
  typedef typename Cx<T>::c C;
  const int parts = p.Dv / p.vc;
  const int node = g / parts, v0 = (g - node * parts) * p.vc;
  constexpr int NW = kThreads / 64;
  const int L = p.L;
  const uint8_t* tau = p.tau + (long long)node * L;
  const int slice = p.Fprev / p.Dv;
  const C* Fin = (const C*)p.F_in + (long long)p.parent[node] * p.Fprev + (long long)v0 * slice;
  C* cur = lds;
  C* nxt = lds + p.gmax;
  auto product = [&](int j, int M) __attribute__((always_inline)) {
    const SmallSite& s = p.site[j];
    const bool last = j == L - 1;
    Product<T> q;
    q.W = (const C*)p.W[j][tau[j] ? 1 : 0] + (last ? v0 * s.dl * s.dd : 0);
    q.N = s.dd * s.dr;
    q.K1 = last ? p.vc : s.du;
    q.K2 = s.dl;
    q.K = q.K1 * q.K2;
    q.M = last ? M : M / s.du;  // [v][u_j][m][r_{j-1}] with m = [u_{j+1} ..][d_0 ..]; the last site sums over v
    q.rows = last ? M : p.vc * q.M;
    return q;
  };
  auto wide = [](const Product<T>& q) { return q.rows >= 32 && q.N >= 32 && q.rows * q.N >= 16 * 256; };
  auto first = [&](const Product<T>& q) __attribute__((always_inline)) {
    const int wave = threadIdx.x >> 6;
    return wide(q) ? load_w<T, 2>(q.W, q.N, q.K, 32 * (wave % ((q.N + 31) / 32)), 0)
                   : load_w<T, 1>(q.W, q.N, q.K, 16 * (wave % ((q.N + 15) / 16)), 0);
  };
  Product<T> q = product(0, slice);
  Chunk<T> wnext = first(q);
  for (int x = threadIdx.x; x < p.vc * slice; x += kThreads) cur[x] = Fin[x];
  __syncthreads();
  for (int j = 0; j < L; ++j) {
    q.A = cur;
    q.C = nxt;
    if (wide(q))
      tiles<T, 2, 2, SPLIT>(q, wnext);
    else if (q.N <= 16 && q.rows >= 64 * NW)
      tiles<T, 4, 1, SPLIT>(q, wnext);
    else
      tiles<T, 1, 1, SPLIT>(q, wnext);
    if (j + 1 < L) {
      q = product(j + 1, q.M * p.site[j].dd);
      wnext = first(q);
    }
    __syncthreads();
    C* t = cur;
    cur = nxt;
    nxt = t;
  }
  // cur: [d_0 ..][d_{L-1}]
  if (parts == 1) {
    small_store<T>(p, node, cur);
  } else {
    C* out = (C*)p.part + (long long)g * p.F;
    for (int x = threadIdx.x; x < p.F; x += kThreads) out[x] = cur[x];
  }
}

// Sum over v of the parts of one node, in order, and the rescale.
template <typename T>
__device__ __forceinline__ void small_sum_body(const SmallRow& p, int node, typename Cx<T>::c* lds) {
  typedef typename Cx<T>::c C;
  const int parts = p.Dv / p.vc;
  const C* part = (const C*)p.part + (long long)node * parts * p.F;
  for (int x = threadIdx.x; x < p.F; x += blockDim.x) {
    C s = {0, 0};
    for (int v0 = 0; v0 < parts; v0 += 8) {  // eight loads in flight
      C q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = v0 + u < parts ? part[(long long)(v0 + u) * p.F + x] : C{0, 0};
#pragma unroll
      for (int u = 0; u < 8; ++u) s += q[u];
    }
    lds[x] = s;
  }
  __syncthreads();
  small_store<T>(p, node, lds);
}

constexpr int kMaxProbs = 32;
struct SmallGroup {
  const SmallRow* probs[kMaxProbs];
  int start[kMaxProbs + 1];
  int nprob;
};

__device__ __forceinline__ int find(const SmallGroup& ga, int g) {
  int lo = 0, hi = ga.nprob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ga.start[mid] <= g) lo = mid; else hi = mid - 1;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

extern __shared__ __attribute__((aligned(16))) char small_lds[];

template <typename T, bool SPLIT>
__global__ __launch_bounds__(kThreads) void small_row(SmallRow p) {
  small_row_body<T, SPLIT>(p, blockIdx.x, (typename Cx<T>::c*)small_lds);
}
template <typename T, bool SPLIT>
__global__ __launch_bounds__(kThreads) void small_row_group(SmallGroup ga) {
  const int i = find(ga, blockIdx.x);
  small_row_body<T, SPLIT>(*ga.probs[i], blockIdx.x - ga.start[i], (typename Cx<T>::c*)small_lds);
}
template <typename T>
__global__ __launch_bounds__(1024) void small_sum(SmallRow p) {
  small_sum_body<T>(p, blockIdx.x, (typename Cx<T>::c*)small_lds);
}
template <typename T>
__global__ __launch_bounds__(1024) void small_sum_group(SmallGroup ga) {
  const int i = find(ga, blockIdx.x);
  small_sum_body<T>(*ga.probs[i], blockIdx.x - ga.start[i], (typename Cx<T>::c*)small_lds);
}

template <typename A>
void go(void (*k)(A), const A& a, int blocks, int threads, size_t lds, hipStream_t st) {
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3((unsigned)threads), lds, st, a);
  hip_check(hipGetLastError(), "small row launch");
}

template <typename A>
void dispatch(void (*ff)(A), void (*fs)(A), void (*fd)(A), const A& a, int prec, int split, int blocks, int threads,
              size_t lds, hipStream_t st) {
  go(prec == PSIM_FP64 ? fd : split ? fs : ff, a, blocks, threads, lds, st);
}

// LDS of a row: its two running-tensor buffers (small_network keeps them in a CU)
size_t row_lds(const SmallRow& p, int eb) { return (size_t)2 * p.gmax * eb; }
int sum_threads(int F) { return F >= 512 ? 1024 : 256; }

}  // namespace

// kind 0: the row itself, 1: the sum over its parts, where a node has several
int small_blocks(const SmallRow& p, int kind) { return p.nodes * (kind == 0 ? p.Dv / p.vc : 1); }
int small_descriptor_bytes() { return (int)sizeof(SmallRow); }

void launch_small(const SmallRow& p, int kind, int prec, int split, void* stream) {
  const int eb = prec == PSIM_FP64 ? 16 : 8;
  if (kind == 0)
    dispatch(small_row<float, false>, small_row<float, true>, small_row<double, false>, p, prec, split,
             small_blocks(p, 0), kThreads, row_lds(p, eb), (hipStream_t)stream);
  else
    dispatch(small_sum<float>, small_sum<float>, small_sum<double>, p, prec, 0, small_blocks(p, 1), sum_threads(p.F),
             (size_t)p.F * eb, (hipStream_t)stream);
}

// Several rows (sums) of one precision and accumulation form: hp the host
// copies, dp their device addresses.
void launch_small_group(const SmallRow* const* hp, const void* const* dp, int n, int kind, int prec, int split,
                        void* stream) {
  const int eb = prec == PSIM_FP64 ? 16 : 8;
  for (int a = 0; a < n; a += kMaxProbs) {
    SmallGroup ga{};
    ga.nprob = std::min(kMaxProbs, n - a);
    size_t lds = 0;
    int fmax = 0;
    int64_t total = 0;
    for (int i = 0; i < ga.nprob; ++i) total += small_blocks(*hp[a + i], kind);
    if (total > 0x7fffffffLL) fail(PSIM_EUNSUPPORTED, "grid too large");
    for (int i = 0; i < ga.nprob; ++i) {
      ga.probs[i] = (const SmallRow*)dp[a + i];
      ga.start[i + 1] = ga.start[i] + small_blocks(*hp[a + i], kind);
      fmax = std::max(fmax, hp[a + i]->F);
      lds = std::max(lds, kind == 0 ? row_lds(*hp[a + i], eb) : (size_t)hp[a + i]->F * eb);
    }
    if (kind == 0)
      dispatch(small_row_group<float, false>, small_row_group<float, true>, small_row_group<double, false>, ga, prec,
               split, ga.start[ga.nprob], kThreads, lds, (hipStream_t)stream);
    else
      dispatch(small_sum_group<float>, small_sum_group<float>, small_sum_group<double>, ga, prec, 0,
               ga.start[ga.nprob], sum_threads(fmax), lds, (hipStream_t)stream);
  }
}

}  // namespace psim
