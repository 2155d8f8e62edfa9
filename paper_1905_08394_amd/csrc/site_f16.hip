// Site contractions of FP32 (4M and 3M) and BF16x3 plans on the 16-bit matrix units.
//
//   C[m][n] = sum_{k1, k2} A[k1][m][k2] * W[k1*K2 + k2][n]        (complex, eq. S4)
//
// Every FP32 operand x (scaled by an exact power of two into the top of the
// half range) is split into two half-precision numbers, x = hi + lo with
// hi = half(x), lo = half(x - hi) (round to nearest even: 22 to 23 significant
// bits), and
//   a b ~= a_hi b_hi + a_hi b_lo + a_lo b_hi
// is accumulated in FP32 by v_mfma_f32_32x32x16_f16: the products are exact
// and the dropped a_lo b_lo is below 2^-22 of the product.  (Error-corrected
// products on matrix units: Ootomo and Yokota, "Recovering single precision
// accuracy from Tensor Cores while surpassing the FP32 theoretical peak
// performance", 2022.)  The complex product is four real ones (Re = ArWr -
// AiWi, Im = ArWi + AiWr).
//
// Why: an FP32 complex multiply-add is 6 (Gauss) or 8 flops on a unit of 157
// TFLOP/s; here it is 24 half flops on a unit 16 times as fast, which sustains
// about 1.1 PFLOP/s (the rate a library half or bfloat16 product of 8192^3
// reaches on this card; the clock falls under that load).  So the floor of a
// contraction is 24 flops per multiply-add at that rate, 46e12 multiply-adds a
// second, or its bytes where K and N are below about 64.
//
// Accuracy: per-instruction sums of 16 products and a last bit less of input
// round the result no more than FP32 instructions of 2 products do.  Error
// (2-norm, against 64 bits) of normal random operands, K = 1024 / 256 / 64:
//   one running sum     5.0e-7 / 2.6e-7 / 1.35e-7   (FP32 4M 8.1e-7 / 4.0e-7 / 2.0e-7, 3M 8.1e-7 / 4.1e-7 / 2.1e-7)
//   partial sums (split) 1.55e-7 / 1.22e-7 / 1.08e-7 (FP32 4M 1.80e-7 / 1.28e-7 / 1.10e-7, 3M 2.15e-7 / 1.74e-7 / 1.28e-7)
// and of amplitudes (rms over seeds): 5x5 (1+32+1) 4M 1.06e-6 -> 0.97e-6, 3M
// 1.10e-6 -> 0.99e-6, 4M split 6.1e-7 -> 5.8e-7, 3M split 7.2e-7 -> 6.0e-7; 5x5
// (1+40+1) 3M split 8.4e-7 -> 6.7e-7; 8x8 (1+25+1) square partition 3M 1.9e-6
// -> 1.5e-6, split 1.29e-6 -> 1.13e-6.
//
// Scale: the halves cover 40 binades, so every node's A is scaled by the
// exponent of its largest component.  A producer on these units measures it
// in its epilogue (amax_out -> amax_in); elsewhere a bound from the last
// rescale is carried along (a_exp: growth_exp(K) per site), which overstates
// the maximum by a few binades and costs no precision until it overstates it by
// about 15.  Components more than 2^-17 below the largest lose relative (not
// absolute) precision: their error stays below 2^-40 of the largest.
//
// Measured (ms before, FP32 units -> now): 16 x (M = 32768, K = N = 1024) split
// 26.3 -> 12.8, unsplit 23.9 -> 11.0; 64 x (4096, 256, 256) split 0.95 -> 0.47,
// unsplit 0.89 -> 0.40; 512 x (4096, 64, 64) split 0.81 -> 0.43 (HBM: 5.0
// TB/s), unsplit 0.68 -> 0.40; 4 x (4096, 4096, 4096) unsplit 12.0 -> 5.7.
//
// BF16x3 is the same kernel with bfloat16 pairs (16 significant bits, the FP32
// range: no scale).  There an instruction sums the Re and Im products of 8 k,
// which is how the real expansion of the complex matrix orders them (kernels.hip,
// the shapes left there), so the results are those of that form bit for bit: a
// last-bit change of an FP32 tensor changes its split, and with it the
// amplitude, by as much as the precision's own error.  5x5 (1+32+1), 256
// bitstrings: interior sites 254 -> 189 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <cstdint>
#include <cstring>

#include "psim_internal.hpp"

namespace psim {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

namespace {

struct F16Args {
  const float* A;
  float* C;
  const float* W0;
  const float* W1;
  const int32_t* a_index;
  const uint8_t* tau;
  const uint32_t* amax_in;   // per node: exponent + 4096 of max |component of A|, 0 = all zeros
  uint32_t* amax_out;
  long long tau_stride;
  long long M, K1, K2, N;
  long long ldw;             // bytes between rows of W
  long long sA_node, sA_v, sC_node, sC_v;
  long long MT, NT, T;
  long long nb, sCw;         // first sites: see GemmLaunch
  long long ldct;            // last sites: row stride of C^T
  int Bz, nst, a_exp, w_exp, beta, stream;
};

constexpr int kTop = 15;     // A is scaled to below 2^kTop,
constexpr int kTopW = 14;    // W below 2^kTopW (both finite as halves)

// One tile: WVM x WVN waves of MBLK x NBLK blocks of 32 x 32 complex outputs.
// Stages of 16 complex k (128-byte rows of A and of W) go global -> LDS
// without registers, double buffered; the other workgroups of the CU cover the
// waits.  A is split in registers as its fragments are read (40 VALU
// instructions for 24 matrix instructions of 32 cycles), so any FP32 tensor
// can be the operand; W was split when it was packed.  Reading W as planes
// (rather than a real expansion of the complex matrix) halves its LDS and L2
// traffic.  SPLIT: the products of each pair of stages are summed apart and
// then added to the running sums.

__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

// The two 16-bit types: vectors, the matrix instruction, and the split of two
// FP32 values (scaled by 2^e) into hi = round(x), lo = round(x - hi).
template <typename H>
struct Half;

template <>
struct Half<_Float16> {
  typedef f16x2 v2;
  typedef f16x8 v8;
  static __device__ __forceinline__ f32x16 mma(v8 a, v8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ v2 round(float a, float b, int e) {
    unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{ldexpf(a, e), ldexpf(b, e)}, v2));
    // hides the packed conversion from the compiler, which otherwise repeats it
    // element by element where the halves are used again
    asm("" : "+v"(u));
    return __builtin_bit_cast(v2, u);
  }
  static __device__ __forceinline__ _Float16 rest(float a, float scale, _Float16 hi) {
    return (_Float16)fmaf(a, scale, -(float)hi);
  }
  static __device__ __forceinline__ void split(float a, float b, int e, float scale, v2& hi, v2& lo) {
    hi = round(a, b, e);
    lo[0] = rest(a, scale, hi[0]);
    lo[1] = rest(b, scale, hi[1]);
  }
};

// bfloat16 has the FP32 range: no scale
template <>
struct Half<__bf16> {
  typedef bf16x2 v2;
  typedef bf16x8 v8;
  static __device__ __forceinline__ f32x16 mma(v8 a, v8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ void split(float a, float b, int, float, v2& hi, v2& lo) {
    hi = __builtin_convertvector(f32x2{a, b}, v2);
    const unsigned u = __builtin_bit_cast(unsigned, hi);
    lo = __builtin_convertvector(f32x2{a - __builtin_bit_cast(float, u << 16),
                                       b - __builtin_bit_cast(float, u & 0xffff0000u)}, v2);
  }
};

// (a, b) pairs to (a, -b) and (b, a)
template <typename V>
__device__ __forceinline__ V conj_pairs(const V x) {
  return __builtin_bit_cast(V, __builtin_bit_cast(u32x4, x) ^ 0x80000000u);
}
template <typename V>
__device__ __forceinline__ V swap_pairs(const V x) {
  u32x4 u = __builtin_bit_cast(u32x4, x);
#pragma unroll
  for (int e = 0; e < 4; ++e) u[e] = __builtin_amdgcn_alignbit(u[e], u[e], 16);
  return __builtin_bit_cast(V, u);
}

template <typename V>
__device__ __forceinline__ V neg(const V x) {
  return __builtin_bit_cast(V, __builtin_bit_cast(u32x4, x) ^ 0x80008000u);
}

// Raises *slot to the exponent + 4096 of the wave's largest m (m >= 0 in every
// lane).  Most waves find it there already and leave the atomic out.
__device__ __forceinline__ void raise_exponent(float m, uint32_t* slot) {
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0 && m > 0) {
    int e;
    frexpf(m, &e);  // m = f 2^e, f in [0.5, 1)
    const uint32_t x = (uint32_t)(e + 4096);
    if (__hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < x) atomicMax(slot, x);
  }
}

// One complex number of an output, past the caches or not.  A launch whose output
// outgrows the 256 MB cache behind the L2s leaves nothing there that its reader
// finds, but pushes out the operands that other tiles share: 5x5 (1+32+1), 256
// bitstrings, FP32 3M 273 -> 262 ms, BF16x3 242 -> 234, 6x6 (1+24+1), 64, 9.35 ->
// 9.02 ms.  Smaller outputs are read from the cache by the next site (6x6
// (1+24+1), 8, BF16x3: 1.30 ms, 1.44 with streaming stores).
template <bool STREAM>
__device__ __forceinline__ void put(float* dst, const f32x2 v) {
  if constexpr (STREAM)
    __builtin_nontemporal_store(v, (f32x2*)dst);
  else
    *(f32x2*)dst = v;
}

#define PSIM_LDS(p) ((__attribute__((address_space(3))) void*)(p))

template <typename H, int WVM, int WVN, int MBLK, int NBLK, bool SPLIT>
__device__ __forceinline__ void site_f16_body(const F16Args& p, const long long t) {
  typedef typename Half<H>::v8 v8;
  constexpr bool PLANAR = __is_same(H, _Float16);  // else bfloat16
  constexpr int NW = WVM * WVN;
  constexpr int BM = WVM * MBLK * 32, BN = WVN * NBLK * 32;
  constexpr int A_INS = BM / 8 / NW, B_INS = BN / 8 / NW;   // wave-wide 1 KB copies (8 rows of 128 bytes)
  static_assert(A_INS >= 1 && B_INS >= 1 && A_INS * NW * 8 == BM && B_INS * NW * 8 == BN, "tile");
  __shared__ __attribute__((aligned(1024))) float sA0[BM * 32];
  __shared__ __attribute__((aligned(1024))) float sA1[BM * 32];
  __shared__ __attribute__((aligned(1024))) float sB0[BN * 32];
  __shared__ __attribute__((aligned(1024))) float sB1[BN * 32];

  const long long nt = t % p.NT;
  const long long rest = t / p.NT;
  const long long mt = rest % p.MT;
  const long long z = rest / p.MT;
  const long long node = z / p.Bz, vb = z % p.Bz;
  const long long ablk = p.a_index ? (long long)p.a_index[node] : node;
  const float* __restrict__ A = p.A + 2 * (ablk * p.sA_node + vb * p.sA_v);
  const int tauv = p.tau ? (int)p.tau[node * p.tau_stride] : 0;
  const char* __restrict__ W = (const char*)(tauv ? p.W1 : p.W0);
  float* __restrict__ C = p.C + 2 * (node * p.sC_node + vb * p.sC_v);
  const long long m0 = mt * BM;
  int sa = 0;
  if (PLANAR) {
    const uint32_t am = p.amax_in ? p.amax_in[node] : 0;
    sa = min(kTop - p.a_exp - (am ? (int)am - 4096 : 0), 127);
  }
  const float scale = ldexpf(1.0f, sa);

  const int tid = threadIdx.x;
  const int lane = tid & 63, wid = tid >> 6;
  const int wr = wid / WVN, wc = wid % WVN;
  const long long sK1 = p.M * p.K2;

  // A stage is 16 complex k: rows of 128 bytes of A and of the packed W
  // (hi / lo halves of Re and Im), 8 chunks of 16 bytes.  Copy `it` of a
  // wave fills tile rows (it * NW + wid) * 8 + lane / 8, physical chunk
  // lane % 8, from logical chunk (lane % 8) ^ swz(row).
  unsigned aoff[A_INS], boff[B_INS];
  const int K2 = (int)p.K2;
#pragma unroll
  for (int it = 0; it < A_INS; ++it) {
    const int row = (it * NW + wid) * 8 + (lane >> 3);
    const int kc = 2 * ((lane & 7) ^ swz(row));   // complex k of the chunk inside the stage
    const long long r = min((long long)row, p.M - 1 - m0);
    const int q = K2 < 16 ? kc / K2 : 0;
    aoff[it] = (unsigned)((q * sK1 + r * K2 + (kc - q * K2)) * 8);
  }
#pragma unroll
  for (int it = 0; it < B_INS; ++it) {
    const int row = (it * NW + wid) * 8 + (lane >> 3);
    const long long r = min((long long)row, p.N - 1 - nt * BN);
    boff[it] = (unsigned)(r * p.ldw) + (unsigned)((lane & 7) ^ swz(row)) * 16u;
  }
  const char* abase = (const char*)(A + 2 * m0 * p.K2);
  const char* bbase = W + nt * BN * p.ldw;
  const long long a_k1 = sK1 * 8 * (K2 < 16 ? 16 / K2 : 1);  // bytes from one k1 step of the stages to the next
  int fk2 = 0;
  auto issue = [&](float* da, float* db) {
#pragma unroll
    for (int it = 0; it < A_INS; ++it)
      __builtin_amdgcn_global_load_lds((const void*)(abase + aoff[it]), PSIM_LDS(da + (it * NW + wid) * 256), 16, 0, 0);
#pragma unroll
    for (int it = 0; it < B_INS; ++it)
      __builtin_amdgcn_global_load_lds((const void*)(bbase + boff[it]), PSIM_LDS(db + (it * NW + wid) * 256), 16, 0, 0);
    bbase += 128;
    fk2 += 16;
    if (fk2 >= K2) {
      abase += a_k1 - (long long)(fk2 - 16) * 8;
      fk2 = 0;
    } else {
      abase += 128;
    }
  };

  f32x16 acc[MBLK][NBLK][2];
#pragma unroll
  for (int bi = 0; bi < MBLK; ++bi)
#pragma unroll
    for (int bj = 0; bj < NBLK; ++bj)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[bi][bj][q][r] = 0;
  f32x16 part[SPLIT ? MBLK : 1][SPLIT ? NBLK : 1][2];

  const int frow = lane & 31, h = lane >> 5;   // lane half h supplies k 8h .. 8h+7 of the stage
  auto compute = [&](const float* as, const float* bs, const bool open, const bool close) {
    if (SPLIT && open) {
#pragma unroll
      for (int bi = 0; bi < MBLK; ++bi)
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj)
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) part[bi][bj][q][r] = 0;
    }
    auto& dst = [&]() -> auto& {
      if constexpr (SPLIT) return part;
      else return acc;
    }();
    // halves: Re hi, Re lo, Im hi, Im lo of the lane's 8 k; bfloat16: hi, lo of
    // Re and Im in turn, of the lane's 4 k of the stage's first and second 8
    v8 w[NBLK][4];
#pragma unroll
    for (int bj = 0; bj < NBLK; ++bj) {
      const int r = (wc * NBLK + bj) * 32 + frow;
      const int sw = swz(r);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = PLANAR ? 2 * q + h : 4 * (q & 1) + 2 * (q >> 1) + h;
        w[bj][q] = *(const v8*)(bs + r * 32 + ((c ^ sw) << 2));
      }
    }
#define PSIM_MM(a, b, c) c = Half<H>::mma(a, b, c)
#pragma unroll
    for (int bi = 0; bi < MBLK; ++bi) {
      const int r = (wr * MBLK + bi) * 32 + frow;
      const int sw = swz(r);
      if constexpr (PLANAR) {
        v8 rh, rl, ih, il;
#pragma unroll
        for (int c = 0; c < 4; ++c) {  // two complex k per chunk
          const f32x4 x = *(const f32x4*)(as + r * 32 + (((4 * h + c) ^ sw) << 2));
          const typename Half<H>::v2 hr = Half<H>::round(x[0], x[2], sa), hi = Half<H>::round(x[1], x[3], sa);
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            rh[2 * c + e] = hr[e];
            ih[2 * c + e] = hi[e];
            rl[2 * c + e] = Half<H>::rest(x[2 * e], scale, hr[e]);
            il[2 * c + e] = Half<H>::rest(x[2 * e + 1], scale, hi[e]);
          }
        }
        const v8 nh = neg(ih), nl = neg(il);
        // Split sums: no instruction moves across the block of products.  Left
        // alone, the scheduler spreads the split of A and the wait for the next
        // stage between them, and each then holds up the products behind it:
        // 5x5 (1+40+1), 16 sharing a prefix, 225 -> 185 ms (0.97 -> 1.2 PFLOP/s);
        // (1+32+1) 3M, 256 bitstrings, 326 -> 287 ms.  Without partial sums three
        // workgroups per CU fill such gaps (6x6 (1+24+1): 11.1 ms, 11.2 fenced).
        if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj) {
          PSIM_MM(rl, w[bj][0], dst[bi][bj][0]);
          PSIM_MM(rl, w[bj][2], dst[bi][bj][1]);
        }
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj) {
          PSIM_MM(nl, w[bj][2], dst[bi][bj][0]);
          PSIM_MM(il, w[bj][0], dst[bi][bj][1]);
        }
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj) {
          PSIM_MM(rh, w[bj][1], dst[bi][bj][0]);
          PSIM_MM(rh, w[bj][3], dst[bi][bj][1]);
        }
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj) {
          PSIM_MM(nh, w[bj][3], dst[bi][bj][0]);
          PSIM_MM(ih, w[bj][1], dst[bi][bj][1]);
        }
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj) {
          PSIM_MM(rh, w[bj][0], dst[bi][bj][0]);
          PSIM_MM(rh, w[bj][2], dst[bi][bj][1]);
        }
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj) {
          PSIM_MM(nh, w[bj][2], dst[bi][bj][0]);
          PSIM_MM(ih, w[bj][0], dst[bi][bj][1]);
        }
        if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int g = 0; g < 2; ++g) {  // 8 k each: an instruction sums their Re and Im products
          v8 xh, xl;
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const f32x4 x = *(const f32x4*)(as + r * 32 + (((4 * g + 2 * h + c) ^ sw) << 2));
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              typename Half<H>::v2 hi, lo;
              Half<H>::split(x[2 * e], x[2 * e + 1], 0, 1.0f, hi, lo);
              xh[4 * c + 2 * e] = hi[0];
              xh[4 * c + 2 * e + 1] = hi[1];
              xl[4 * c + 2 * e] = lo[0];
              xl[4 * c + 2 * e + 1] = lo[1];
            }
          }
          // (Re, -Im) for Re C, (Im, Re) for Im C
          const v8 ph = conj_pairs(xh), pl = conj_pairs(xl), qh = swap_pairs(xh), ql = swap_pairs(xl);
#pragma unroll
          for (int bj = 0; bj < NBLK; ++bj) {
            PSIM_MM(pl, w[bj][2 * g], dst[bi][bj][0]);
            PSIM_MM(ql, w[bj][2 * g], dst[bi][bj][1]);
          }
#pragma unroll
          for (int bj = 0; bj < NBLK; ++bj) {
            PSIM_MM(ph, w[bj][2 * g + 1], dst[bi][bj][0]);
            PSIM_MM(qh, w[bj][2 * g + 1], dst[bi][bj][1]);
          }
#pragma unroll
          for (int bj = 0; bj < NBLK; ++bj) {
            PSIM_MM(ph, w[bj][2 * g], dst[bi][bj][0]);
            PSIM_MM(qh, w[bj][2 * g], dst[bi][bj][1]);
          }
        }
      }
    }
#undef PSIM_MM
    if (SPLIT && close) {
#pragma unroll
      for (int bi = 0; bi < MBLK; ++bi)
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj)
#pragma unroll
          for (int q = 0; q < 2; ++q) acc[bi][bj][q] += part[bi][bj][q];
    }
  };
  constexpr unsigned kWaitVm0 = 0x3f70;  // vmcnt(0), other counters unconstrained

  issue(sA0, sB0);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __syncthreads();
  const int nst = p.nst;
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    issue(sA1, sB1);
    compute(sA0, sB0, true, false);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    if (s + 2 < nst) issue(sA0, sB0);
    compute(sA1, sB1, false, true);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
  }
  if (s < nst) compute(sA0, sB0, true, true);

  const int sc = PLANAR ? p.w_exp - sa - kTopW : p.w_exp;
  float mx = 0;
  auto store = [&](auto stream) {
#pragma unroll
    for (int bi = 0; bi < MBLK; ++bi)
#pragma unroll
      for (int bj = 0; bj < NBLK; ++bj)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const long long row = m0 + (wr * MBLK + bi) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
          const long long col = nt * BN + (wc * NBLK + bj) * 32 + frow;
          if (row < p.M && col < p.N) {
            const f32x2 v = {ldexpf(acc[bi][bj][0][r], sc), ldexpf(acc[bi][bj][1][r], sc)};
            mx = fmaxf(mx, fmaxf(fabsf(v[0]), fabsf(v[1])));
            put<stream.value>(C + 2 * (row * p.N + col), v);
          }
        }
  };
  if (p.stream)
    store(std::true_type{});
  else
    store(std::false_type{});
  if (p.amax_out) raise_exponent(mx, p.amax_out + node);
}

template <typename H, int WVM, int WVN, int MBLK, int NBLK, bool SPLIT, int OCC>
__global__ __launch_bounds__(64 * WVM * WVN, OCC) void site_f16(F16Args p) {
  // XCD-aware order: workgroup b runs on XCD b mod 8; each XCD gets a contiguous range of tiles
  const long long per_xcd = (p.T + 7) / 8;
  const long long t = (long long)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= p.T) return;
  site_f16_body<H, WVM, WVN, MBLK, NBLK, SPLIT>(p, t);
}

// Several contractions in one grid: problem i owns tiles [start[i],
// start[i+1]), its arguments lie in device memory.
constexpr int kMaxProbs = 32;
struct F16Group {
  const F16Args* probs[kMaxProbs];
  long long start[kMaxProbs + 1];
  int nprob;
};

// The problem that owns this workgroup's tile and its number there, or -1.
__device__ __forceinline__ long long group_tile(const F16Group& ga, F16Args& p) {
  const long long total = ga.start[ga.nprob];
  const long long per_xcd = (total + 7) / 8;
  const long long g = (long long)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (g >= total) return -1;
  int lo = 0, hi = ga.nprob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ga.start[mid] <= g) lo = mid; else hi = mid - 1;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const int* src = (const int*)ga.probs[lo];
  int* dst = (int*)&p;
#pragma unroll
  for (int w = 0; w < (int)(sizeof(F16Args) / 4); ++w) dst[w] = __builtin_amdgcn_readfirstlane(src[w]);
  return g - ga.start[lo];
}

template <typename H, int WVM, int WVN, int MBLK, int NBLK, bool SPLIT, int OCC>
__global__ __launch_bounds__(64 * WVM * WVN, OCC) void site_f16_group(F16Group ga) {
  F16Args p;
  const long long t = group_tile(ga, p);
  if (t >= 0) site_f16_body<H, WVM, WVN, MBLK, NBLK, SPLIT>(p, t);
}

// First sites of a row (K2 = 1, A[k][m]): FP32 products, FP32 sums, for every
// precision but FP64.  Each output takes few products (K = one bond) and the
// output is the row's largest tensor, so the time is that of writing it.  An A
// stage (8 k of 128 m, 1 KB each) goes to LDS as it lies and is read with m
// across the lanes; Re and Im have an accumulator each, so a lane stores whole
// complex numbers, 256 bytes to a row.  The K-major form of the general kernel
// turned A round on its way through registers with conflicting 4-byte LDS
// stores and wrote 4 bytes a lane.  The products and their order are that
// form's (4M): the results are the same bit for bit.
// 5x5 (1+32+1), 256 bitstrings: BF16x3 52 -> 25 ms, FP32 3M 30 -> 25 (about 100
// GB written: 4 TB/s); 6x6 (1+24+1) 2.6 -> 1.0 ms; bond 32 (K = 32, 5x5
// (1+40+1)) 2.98 -> 3.01 ms a launch, where the products take as long as the
// writes.
template <bool SPLIT>
__device__ __forceinline__ void site_first_body(const F16Args& p, const long long t) {
  constexpr int BM = 128, BN = 64, BK = 8;
  __shared__ __attribute__((aligned(1024))) float sA0[BM * BK * 2], sA1[BM * BK * 2];
  __shared__ __attribute__((aligned(1024))) float sB0[BN * BK * 2], sB1[BN * BK * 2];

  const long long nt = t % p.NT;
  const long long rest = t / p.NT;
  const long long mt = rest % p.MT;
  const long long z = rest / p.MT;
  const long long node = z / p.Bz, vb = z % p.Bz;
  const long long ablk = p.a_index ? (long long)p.a_index[node] : node;
  const float* __restrict__ A = p.A + 2 * (ablk * p.sA_node + vb * p.sA_v);
  const int tauv = p.tau ? (int)p.tau[node * p.tau_stride] : 0;
  const char* __restrict__ W = (const char*)(tauv ? p.W1 : p.W0);
  float* __restrict__ C = p.C + 2 * (node * p.sC_node + vb * p.sC_v);
  const long long m0 = mt * BM, n0 = nt * BN;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;

  // A: wave copy `it` is row 4 it + wid of the stage, two m per lane (M even).
  // W: rows of 64 bytes (8 complex k), 16 rows per wave, physical chunk lane % 4
  // from logical (lane % 4) ^ (row / 2) % 4.
  const char* a_src = (const char*)(A + 2 * (wid * p.M + min(m0 + 2 * lane, p.M - 2)));
  const int brow = wid * 16 + (lane >> 2);
  const char* b_src = W + min(n0 + brow, p.N - 1) * p.ldw + (((lane & 3) ^ (brow >> 1)) & 3) * 16;
  const long long a_step = 4 * p.M * 8;
  auto issue = [&](float* da, float* db) {
    __builtin_amdgcn_global_load_lds((const void*)a_src, PSIM_LDS(da + wid * 256), 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void*)(a_src + a_step), PSIM_LDS(da + (4 + wid) * 256), 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void*)b_src, PSIM_LDS(db + wid * 256), 16, 0, 0);
    a_src += 2 * a_step;
    b_src += 64;
  };

  f32x16 acc[2][2], part[SPLIT ? 2 : 1][2];
#pragma unroll
  for (int bj = 0; bj < 2; ++bj)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[bj][q][r] = 0;

  const int frow = lane & 31, h = lane >> 5;
  // open, close: first and last stage of a partial sum (16 k)
  auto compute = [&](const float* as, const float* bs, const bool open, const bool close) {
    if (SPLIT && open) {
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int r = 0; r < 16; ++r) part[SPLIT ? bj : 0][q][r] = 0;
    }
    auto& dst = [&]() -> auto& {
      if constexpr (SPLIT) return part;
      else return acc;
    }();
#pragma unroll
    for (int g = 0; g < BK / 4; ++g) {  // lane half h: k 4g + 2h and the next
      f32x2 a[2];
      f32x4 w[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) a[c] = *(const f32x2*)(as + (4 * g + 2 * h + c) * 256 + 2 * (wid * 32 + frow));
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const int r = bj * 32 + frow;
        w[bj] = *(const f32x4*)(bs + r * 16 + (((2 * g + h) ^ (r >> 1)) & 3) * 4);
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
          dst[bj][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][0], w[bj][2 * c], dst[bj][0], 0, 0, 0);
          dst[bj][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][0], w[bj][2 * c + 1], dst[bj][1], 0, 0, 0);
        }
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
          dst[bj][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][1], -w[bj][2 * c + 1], dst[bj][0], 0, 0, 0);
          dst[bj][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[c][1], w[bj][2 * c], dst[bj][1], 0, 0, 0);
        }
      }
    }
    if (SPLIT && close) {
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[bj][q] += part[SPLIT ? bj : 0][q];
    }
  };
  constexpr unsigned kWaitVm0 = 0x3f70;

  issue(sA0, sB0);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __syncthreads();
  const int nst = p.nst;
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    issue(sA1, sB1);
    compute(sA0, sB0, true, false);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    if (s + 2 < nst) issue(sA0, sB0);
    compute(sA1, sB1, false, true);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
  }
  if (s < nst) compute(sA0, sB0, true, true);

  auto store = [&](auto stream) {
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const long long col = n0 + bj * 32 + frow;
      if (col >= p.N) continue;
      // plain rows, or blocks of nb columns
      float* dst = C + 2 * (p.nb ? (col / p.nb) * p.sCw + col % p.nb : col);
      const long long ld = p.nb ? p.nb : p.N;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const long long row = m0 + wid * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (row < p.M) put<stream.value>(dst + 2 * row * ld, f32x2{acc[bj][0][r], acc[bj][1][r]});
      }
    }
  };
  if (p.stream)
    store(std::true_type{});
  else
    store(std::false_type{});
}

template <bool SPLIT>
__global__ __launch_bounds__(256, SPLIT ? 3 : 4) void site_first(F16Args p) {
  const long long per_xcd = (p.T + 7) / 8;
  const long long t = (long long)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t < p.T) site_first_body<SPLIT>(p, t);
}

template <bool SPLIT>
__global__ __launch_bounds__(256, SPLIT ? 3 : 4) void site_first_group(F16Group ga) {
  F16Args p;
  const long long t = group_tile(ga, p);
  if (t >= 0) site_first_body<SPLIT>(p, t);
}

// Last sites of a row (transposed stores, up to 32 output columns): FP32 4M
// products on the real expansion of W.  The row's largest tensor is read once
// and its result is small, so the time is that of reading it, if no matrix
// instruction works on padding: tiles are 32 NBLK reals (16 or 32 complex
// columns) wide, 128 m high, one wave to 32 m.  A and W stages (rows of 16
// complex k) go to LDS without registers.  The blocks hold C^T, so lanes run
// along m and store whole complex numbers.  Products and order are those of the
// general kernel: the results are the same bit for bit.
// 5x5 (1+32+1), 256 bitstrings: 30 -> 22 ms (100 GB read: 4.6 TB/s); 6x6
// (1+24+1) 1.4 -> 1.0 ms; 32 columns (bond 32, 5x5 (1+40+1)) 7.7 -> 6.8 ms.
template <int NBLK, bool SPLIT>
__global__ __launch_bounds__(256, NBLK == 1 ? 4 : 3) void site_last(F16Args p) {
  constexpr int BM = 128, BN = 32 * NBLK;
  __shared__ __attribute__((aligned(1024))) float sA0[BM * 32], sA1[BM * 32];
  __shared__ __attribute__((aligned(1024))) float sB0[BN * 32], sB1[BN * 32];

  const long long per_xcd = (p.T + 7) / 8;
  const long long t = (long long)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= p.T) return;
  const long long mt = t % p.MT;
  const long long z = t / p.MT;
  const long long node = z / p.Bz, vb = z % p.Bz;
  const long long ablk = p.a_index ? (long long)p.a_index[node] : node;
  const float* __restrict__ A = p.A + 2 * (ablk * p.sA_node + vb * p.sA_v);
  const int tauv = p.tau ? (int)p.tau[node * p.tau_stride] : 0;
  const char* __restrict__ W = (const char*)(tauv ? p.W1 : p.W0);
  float* __restrict__ C = p.C + 2 * (node * p.sC_node + vb * p.sC_v);
  const long long m0 = mt * BM;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const long long sK1 = p.M * p.K2;
  const int K2 = (int)p.K2;

  // copies as in site_f16_body; W rows past the last column repeat it
  unsigned aoff[4], boff[NBLK];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = (it * 4 + wid) * 8 + (lane >> 3);
    const int kc = 2 * ((lane & 7) ^ swz(row));
    const long long r = min((long long)row, p.M - 1 - m0);
    const int q = K2 < 16 ? kc / K2 : 0;
    aoff[it] = (unsigned)((q * sK1 + r * K2 + (kc - q * K2)) * 8);
  }
#pragma unroll
  for (int it = 0; it < NBLK; ++it) {
    const int row = (it * 4 + wid) * 8 + (lane >> 3);
    boff[it] = (unsigned)(min((long long)row, 2 * p.N - 1) * p.ldw) + (unsigned)((lane & 7) ^ swz(row)) * 16u;
  }
  const char* abase = (const char*)(A + 2 * m0 * p.K2);
  const char* bbase = W;
  const long long a_k1 = sK1 * 8 * (K2 < 16 ? 16 / K2 : 1);
  int fk2 = 0;
  auto issue = [&](float* da, float* db) {
#pragma unroll
    for (int it = 0; it < 4; ++it)
      __builtin_amdgcn_global_load_lds((const void*)(abase + aoff[it]), PSIM_LDS(da + (it * 4 + wid) * 256), 16, 0, 0);
#pragma unroll
    for (int it = 0; it < NBLK; ++it)
      __builtin_amdgcn_global_load_lds((const void*)(bbase + boff[it]), PSIM_LDS(db + (it * 4 + wid) * 256), 16, 0, 0);
    bbase += 128;
    fk2 += 16;
    if (fk2 >= K2) {
      abase += a_k1 - (long long)(fk2 - 16) * 8;
      fk2 = 0;
    } else {
      abase += 128;
    }
  };

  f32x16 acc[NBLK];
#pragma unroll
  for (int bj = 0; bj < NBLK; ++bj)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[bj][r] = 0;
  const int frow = lane & 31, h = lane >> 5;
  auto compute = [&](const float* as, const float* bs) {
    f32x16 part[SPLIT ? NBLK : 1];
    if (SPLIT) {
#pragma unroll
      for (int bj = 0; bj < NBLK; ++bj)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[SPLIT ? bj : 0][r] = 0;
    }
    auto& dst = [&]() -> auto& {
      if constexpr (SPLIT) return part;
      else return acc;
    }();
#pragma unroll
    for (int g = 0; g < 4; ++g) {  // 8 reals: lane half h reads 8g + 4h .. 8g + 4h + 3
      const int ra = wid * 32 + frow;
      const f32x4 a = *(const f32x4*)(as + ra * 32 + (((2 * g + h) ^ swz(ra)) << 2));
      f32x4 w[NBLK];
#pragma unroll
      for (int bj = 0; bj < NBLK; ++bj) {
        const int r = bj * 32 + frow;
        w[bj] = *(const f32x4*)(bs + r * 32 + (((2 * g + h) ^ swz(r)) << 2));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int bj = 0; bj < NBLK; ++bj)
          dst[bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[bj][e], a[e], dst[bj], 0, 0, 0);
    }
    if (SPLIT) {
#pragma unroll
      for (int bj = 0; bj < NBLK; ++bj) acc[bj] += part[SPLIT ? bj : 0];
    }
  };
  constexpr unsigned kWaitVm0 = 0x3f70;

  issue(sA0, sB0);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __syncthreads();
  const int nst = p.nst;
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    issue(sA1, sB1);
    compute(sA0, sB0);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    if (s + 2 < nst) issue(sA0, sB0);
    compute(sA1, sB1);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
  }
  if (s < nst) compute(sA0, sB0);

  const long long m = m0 + wid * 32 + frow;
  if (m >= p.M) return;
#pragma unroll
  for (int bj = 0; bj < NBLK; ++bj)
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const int n = (bj * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) >> 1;
      if (n >= p.N) continue;
      f32x2* dst = (f32x2*)(C + 2 * (n * p.ldct + m));
      f32x2 v = {acc[bj][r], acc[bj][r + 1]};
      if (p.beta) v += *dst;
      *dst = v;
    }
}

// Packed FP32 rows (Re, Im interleaved along k, groups of 16 complex k = 128
// bytes) to halves of the same 16 k, scaled by 2^kTopW: Re hi, Re lo, Im hi, Im
// lo; or to bfloat16: all hi, all lo, Re and Im in turn.  One thread per group,
// so src and dst may be the same.
template <typename H>
__global__ void pack_w_f16(const float* src, float* dst, long long groups) {
  typedef typename Half<H>::v8 v8;
  constexpr bool planar = __is_same(H, _Float16);
  constexpr int e = planar ? kTopW : 0;
  for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < groups;
       g += (long long)gridDim.x * blockDim.x) {
    f32x4 x[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) x[c] = *(const f32x4*)(src + 32 * g + 4 * c);
    v8 o[8];
#pragma unroll
    for (int k = 0; k < 16; k += 2)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4 v = x[k >> 1];
        typename Half<H>::v2 hi, lo;
        if (planar)  // Re (q = 0) or Im of k, k + 1
          Half<H>::split(v[q], v[2 + q], e, ldexpf(1.0f, e), hi, lo);
        else         // Re, Im of k + q
          Half<H>::split(v[2 * q], v[2 * q + 1], e, 1.0f, hi, lo);
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const int ch = planar ? 4 * q + (k >> 3) : k >> 2, at = planar ? (k & 7) + d : 2 * ((k & 3) + q) + d;
          o[ch][at] = hi[d];
          o[ch + (planar ? 2 : 4)][at] = lo[d];
        }
      }
#pragma unroll
    for (int c = 0; c < 8; ++c) *(v8*)(dst + 32 * g + 4 * c) = o[c];
  }
}

// Exponent + 4096 of the largest component of each node's tensor (out zeroed before).
__global__ __launch_bounds__(256) void exponents_f16(const float* __restrict__ A, long long len, long long stride,
                                                     uint32_t* out) {
  const float* a = A + (long long)blockIdx.y * stride;
  float m = 0;
  // infinities and NaN stay out: they must not set the scale of the finite rows
  auto take = [&](float v) {
    v = fabsf(v);
    if (v < __builtin_inff()) m = fmaxf(m, v);
  };
  for (long long x = (long long)blockIdx.x * 256 + threadIdx.x; 4 * x + 3 < len; x += (long long)gridDim.x * 256) {
    const f32x4 v = *(const f32x4*)(a + 4 * x);
#pragma unroll
    for (int e = 0; e < 4; ++e) take(v[e]);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0)
    for (long long x = len / 4 * 4; x < len; ++x) take(a[x]);
  raise_exponent(m, out + blockIdx.y);
}

}  // namespace

void launch_pack_w_f16(const void* src, void* dst, int64_t groups, void* stream, bool bf16) {
  const long long b = std::max<long long>(1, std::min<long long>((groups + 255) / 256, 1 << 16));
  hipLaunchKernelGGL(bf16 ? pack_w_f16<__bf16> : pack_w_f16<_Float16>, dim3((unsigned)b), dim3(256), 0,
                     (hipStream_t)stream, (const float*)src, (float*)dst, (long long)groups);
  hip_check(hipGetLastError(), "pack_w_f16 launch");
}

void launch_exponents_f16(const void* A, int64_t per_node, int64_t stride, int64_t nodes, uint32_t* out, void* stream) {
  launch_zero_u32(out, nodes, stream);
  const long long gx = std::max<long long>(1, std::min<long long>((2 * per_node + 4095) / 4096, 2048));
  for (int64_t n0 = 0; n0 < nodes; n0 += 65535) {
    const int64_t n = std::min<int64_t>(65535, nodes - n0);
    hipLaunchKernelGGL(exponents_f16, dim3((unsigned)gx, (unsigned)n), dim3(256), 0, (hipStream_t)stream,
                       (const float*)A + 2 * n0 * stride, (long long)(2 * per_node), (long long)(2 * stride), out + n0);
  }
  hip_check(hipGetLastError(), "exponents_f16 launch");
}

// Stages of 16 complex k: inside one k1 block (K2 a multiple of 16) or whole
// k1 blocks (K2 = 2, 4, 8), read as 16-byte chunks (K2 even).  The copies'
// offsets from a stage's base are 32-bit: 128 rows of A, and for a small K2
// 16 / K2 blocks of M rows.
bool f16_site(int prec, int64_t M, int64_t K1, int64_t K2) {
  return prec != PSIM_FP64 && K2 % 2 == 0 && (K1 * K2) % 16 == 0 &&
         (K2 % 16 == 0 || 16 % K2 == 0) && (K2 < 16 ? M < (1 << 24) : K2 < (1 << 21)) && K1 * K2 < (1 << 21);
}

// Whole stages of 8 k, read as 16-byte chunks of two m.
bool first_site(int prec, int64_t M, int64_t K1, int64_t K2) {
  return prec != PSIM_FP64 && K2 == 1 && K1 % 8 == 0 && M % 2 == 0 && K1 < (1 << 21);
}

// Tiles: every form has the same products in the same order for each output.
//   0: 128 x 128 complex outputs, 4 waves of 64 x 64, two workgroups per CU
//   1: 128 x 64, 4 waves of 32 x 64, three workgroups per CU
//   2: the same with partial sums, two workgroups per CU
//   3, 4: 0 and 1 for BF16x3
//   5, 6: first sites, 128 x 64, without and with partial sums (up to 16 k there
//   is one partial sum, the result itself)
static int f16_variant(const GemmLaunch& g) {
  if (g.f16 == 3) return g.split && g.K1 > 16 ? 6 : 5;
  if (g.split && g.f16 == 1) return 2;
  const long long big = ((g.M + 127) / 128) * ((g.N + 127) / 128) * g.nodes * g.Bz;
  return (g.N % 128 == 0 && big >= 1024 ? 0 : 1) + (g.f16 == 2 ? 3 : 0);
}

static F16Args f16_args(const GemmLaunch& g, int variant) {
  if (g.M < 1 || g.K1 < 1 || g.K2 < 1 || g.N < 1 || g.nodes < 1 || g.Bz < 1)
    fail(PSIM_EINVAL, "site gemm: non-positive size");
  const bool first = g.f16 == 3;
  if (!(first ? first_site(g.prec, g.M, g.K1, g.K2) : !g.nb && f16_site(g.prec, g.M, g.K1, g.K2)) || g.trans_out || g.beta || (uintptr_t)g.A % 16 || g.sA_node % 2 ||
      g.sA_v % 2 || g.ldw >= (1 << 23))
    fail(PSIM_EINTERNAL, "site gemm: shape or alignment the half-precision kernels do not take");
  F16Args a{};
  a.A = (const float*)g.A;
  a.C = (float*)g.C;
  a.W0 = (const float*)g.W0;
  a.W1 = (const float*)(g.W1 ? g.W1 : g.W0);
  a.a_index = g.a_index;
  a.tau = g.tau;
  a.tau_stride = g.tau_stride;
  a.amax_in = g.amax_in;
  a.amax_out = g.amax_out;
  a.M = g.M;
  a.K1 = g.K1;
  a.K2 = g.K2;
  a.N = g.N;
  a.ldw = g.ldw * 4;
  a.sA_node = g.sA_node;
  a.sA_v = g.sA_v;
  a.sC_node = g.sC_node;
  a.sC_v = g.sC_v;
  a.Bz = g.Bz;
  a.stream = g.M * g.N * g.nodes * g.Bz > (1 << 25);  // 256 MB of complex64
  a.nb = g.nb;
  a.sCw = g.sCw;
  a.nst = (int)(g.K1 * g.K2 / (first ? 8 : 16));
  a.a_exp = g.a_exp;
  a.w_exp = g.w_exp;
  const int bn = variant == 0 || variant == 3 ? 128 : 64;
  a.MT = (a.M + 127) / 128;
  a.NT = (a.N + bn - 1) / bn;
  a.T = a.MT * a.NT * g.nodes * g.Bz;
  return a;
}

void launch_site_f16(const GemmLaunch& g, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int variant = f16_variant(g);
  const F16Args a = f16_args(g, variant);
  const long long blocks = (a.T + 7) / 8 * 8;
  if (blocks > 0x7fffffffLL) fail(PSIM_EUNSUPPORTED, "grid too large");
  const dim3 grid((unsigned)blocks), wg(256);
  switch (variant) {
    case 0: hipLaunchKernelGGL((site_f16<_Float16, 2, 2, 2, 2, false, 2>), grid, wg, 0, st, a); break;
    case 1: hipLaunchKernelGGL((site_f16<_Float16, 4, 1, 1, 2, false, 3>), grid, wg, 0, st, a); break;
    case 2: hipLaunchKernelGGL((site_f16<_Float16, 4, 1, 1, 2, true, 2>), grid, wg, 0, st, a); break;
    case 3: hipLaunchKernelGGL((site_f16<__bf16, 2, 2, 2, 2, false, 2>), grid, wg, 0, st, a); break;
    case 4: hipLaunchKernelGGL((site_f16<__bf16, 4, 1, 1, 2, false, 3>), grid, wg, 0, st, a); break;
    case 5: hipLaunchKernelGGL((site_first<false>), grid, wg, 0, st, a); break;
    default: hipLaunchKernelGGL((site_first<true>), grid, wg, 0, st, a); break;
  }
  hip_check(hipGetLastError(), "site_f16 launch");
}

// The stages are f16_site's, the columns fit one tile, and every 16-byte copy is
// aligned.
bool last_site(const GemmLaunch& g) {
  return g.trans_out && g.N <= 32 && g.prec != PSIM_FP32_3M && f16_site(g.prec, g.M, g.K1, g.K2) &&
         (uintptr_t)g.A % 16 == 0 && g.sA_node % 2 == 0 && g.sA_v % 2 == 0 && g.w_koff % 2 == 0 && g.ldw < (1 << 23) && !g.nb;
}

void launch_site_last(const GemmLaunch& g, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  F16Args a{};
  a.A = (const float*)g.A;
  a.C = (float*)g.C;
  a.W0 = (const float*)g.W0 + 2 * g.w_koff;
  a.W1 = (const float*)(g.W1 ? g.W1 : g.W0) + 2 * g.w_koff;
  a.a_index = g.a_index;
  a.tau = g.tau;
  a.tau_stride = g.tau_stride;
  a.M = g.M;
  a.K2 = g.K2;
  a.N = g.N;
  a.ldw = g.ldw * 4;
  a.sA_node = g.sA_node;
  a.sA_v = g.sA_v;
  a.sC_node = g.sC_node;
  a.sC_v = g.sC_v;
  a.ldct = g.ldct ? g.ldct : g.M;
  a.beta = g.beta;
  a.Bz = g.Bz;
  a.nst = (int)(g.K1 * g.K2 / 16);
  a.MT = (a.M + 127) / 128;
  a.T = a.MT * g.nodes * g.Bz;
  const long long blocks = (a.T + 7) / 8 * 8;
  if (blocks > 0x7fffffffLL) fail(PSIM_EUNSUPPORTED, "grid too large");
  const dim3 grid((unsigned)blocks), wg(256);
  if (g.N <= 16)
    hipLaunchKernelGGL((g.split ? site_last<1, true> : site_last<1, false>), grid, wg, 0, st, a);
  else
    hipLaunchKernelGGL((g.split ? site_last<2, true> : site_last<2, false>), grid, wg, 0, st, a);
  hip_check(hipGetLastError(), "site_last launch");
}

int f16_descriptor_bytes() { return (int)sizeof(F16Args); }

int group_variant_f16(const GemmLaunch& g, void* out, long long* tiles) {
  const int variant = f16_variant(g);
  const F16Args a = f16_args(g, variant);
  std::memcpy(out, &a, sizeof(a));
  *tiles = a.T;
  return variant;
}

void launch_group_f16(int variant, const void* const* d_probs, const long long* start, int nprob, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (nprob < 1 || nprob > kMaxProbs || variant < 0 || variant > 6) fail(PSIM_EINTERNAL, "bad f16 group");
  F16Group ga{};
  for (int i = 0; i < nprob; ++i) {
    ga.probs[i] = (const F16Args*)d_probs[i];
    ga.start[i] = start[i];
  }
  ga.start[nprob] = start[nprob];
  ga.nprob = nprob;
  if (start[nprob] < 1) return;
  const long long blocks = (start[nprob] + 7) / 8 * 8;
  if (blocks > 0x7fffffffLL) fail(PSIM_EUNSUPPORTED, "grid too large");
  const dim3 grid((unsigned)blocks), wg(256);
  switch (variant) {
    case 0: hipLaunchKernelGGL((site_f16_group<_Float16, 2, 2, 2, 2, false, 2>), grid, wg, 0, st, ga); break;
    case 1: hipLaunchKernelGGL((site_f16_group<_Float16, 4, 1, 1, 2, false, 3>), grid, wg, 0, st, ga); break;
    case 2: hipLaunchKernelGGL((site_f16_group<_Float16, 4, 1, 1, 2, true, 2>), grid, wg, 0, st, ga); break;
    case 3: hipLaunchKernelGGL((site_f16_group<__bf16, 2, 2, 2, 2, false, 2>), grid, wg, 0, st, ga); break;
    case 4: hipLaunchKernelGGL((site_f16_group<__bf16, 4, 1, 1, 2, false, 3>), grid, wg, 0, st, ga); break;
    case 5: hipLaunchKernelGGL((site_first_group<false>), grid, wg, 0, st, ga); break;
    default: hipLaunchKernelGGL((site_first_group<true>), grid, wg, 0, st, ga); break;
  }
  hip_check(hipGetLastError(), "grouped site_f16 launch");
}

}  // namespace psim
