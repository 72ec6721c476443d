// Coulomb matrix through the n^3 Chebyshev grid tensor, B never formed
// (eq. coulapprox with the mode products of eq. ig1), FP64:
//
//   Dt_q       = D(k,l) (2 - delta_kl)                     q = (k,l), k <= l
//   rho(a)     = sum_q Dt_q m_{q,0}(a0) m_{q,1}(a1) m_{q,2}(a2)
//   Phi        = (2/sqrt(pi)) sum_k w_k  rho x_0 K_k x_1 K_k x_2 K_k
//   J_p        = sum_a m_{p,0}(a0) m_{p,1}(a1) m_{p,2}(a2) Phi(a)
//   J(mu,nu)   = J(nu,mu) = J_p,                           p = (mu,nu)
//
// Both pair contractions run on the FP64 matrix cores (v_mfma_f64_16x16x4):
//  * rho: for each a0, rho_a0 = (c_a0 o M_1) M_2^T with c_a0(q) = Dt_q m_{q,0}(a0),
//    an n x n product over the pairs.  A work group owns 8 or 16 values of a0
//    and one chunk of pairs, stages the chunk's moments in LDS 64 pairs at a
//    time (loads for the next batch in flight during the MFMAs) and writes an
//    n^3 partial; the partials are summed in a fixed order, so the result does
//    not depend on scheduling.
//  * J_p: for a tile of 16 pairs, X(a0, a1, p) = sum_a2 Phi(a0, a1, a2) m_{p,2}(a2)
//    is an MFMA product with Phi staged in LDS one a0 slab at a time; the
//    output fragment is contracted at once with m_{p,1} (in registers) and
//    m_{p,0}, so X is never stored.
#include "tai_internal.h"
#include "tai_device.h"

#include <algorithm>
#include <type_traits>

namespace tai {
namespace {

constexpr double kTwoOverSqrtPi = 1.1283791670955126;

// Pair p of the moments is pair pairs[p] of the full list when a screened
// list is given (entries outside the full list contribute nothing).
__device__ inline bool pair_of(const int32_t* pairs, int nb, int64_t p, int& mu, int& nu) {
  int64_t g = p;
  if (pairs) {
    g = pairs[p];
    if (g < 0 || g >= (int64_t)nb * (nb + 1) / 2) return false;
  }
  decode_pair(nb, g, mu, nu);
  return true;
}

// Pair densities; the first work group also writes out[i] = scale w[i % nq] for
// i < nq reps: the quadrature weights, repeated for each source box of the adaptive
// J, with 2/sqrt(pi) folded in (a launch of their own was 2.3 us).
struct ScaledWeights {
  const double* w;
  int nq, reps;
  double scale;
  double* out;
};
__global__ void __launch_bounds__(256)
density_pairs_kernel(const double* __restrict__ D, int nb, int64_t npair, const int32_t* __restrict__ pairs,
                     double* __restrict__ Dt, ScaledWeights sw) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < sw.nq * sw.reps; i += blockDim.x) sw.out[i] = sw.scale * sw.w[i % sw.nq];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npair) return;
  int mu, nu;
  Dt[p] = pair_of(pairs, nb, p, mu, nu) ? D[(int64_t)mu * nb + nu] * (mu == nu ? 1.0 : 2.0) : 0.0;
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kKB = 64;          // pairs per LDS batch of the rho kernel
constexpr int kRhoGroups = 512;  // target work groups of the rho kernel

// The arithmetic of the two pair contractions: FP64, or FP32 with the
// products summed in FP32 within one LDS batch of pairs (rho) or one a1
// block (J_p) and in FP64 beyond.  Both use 16x16x4 MFMAs, whose operand
// fragments have the same lane layout; the output rows differ (row_of).
struct JF64 {
  using T = double;
  using Acc = v4d;
  static constexpr bool kSplitSum = false;
  __device__ static Acc mma(double a, double b, Acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row_of(int kg, int r) { return kg + 4 * r; }
};
struct JF32 {
  using T = float;
  using Acc = v4f;
  static constexpr bool kSplitSum = true;
  __device__ static Acc mma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row_of(int kg, int r) { return 4 * kg + r; }
};

// Shapes of the rho kernel.  A work group of eight waves owns A0G values of a0
// and one chunk of pairs; a wave owns A0W values of a0 and all (a1, a2), as
// RT x NT output tiles of 16 x 16 over the packed rows (a0, a1):
//   HALF: n <= 16 NT - 8 and A0W = 2.  Two values of a0 fill 2 NT - 1 blocks of
// rows instead of 2 NT.
//   KS = 2: waves w and w + 4 share their values of a0 and take half of each
// batch's pairs, their sums added at the end.  Half the values of a0 per work
// group: twice the work groups for short pair lists, and no padding to 16
// values of a0 at n = 24 or 40.
template <int NT_, int A0W_, bool HALF_, int KS_>
struct RhoShape {
  static constexpr int NT = NT_, A0W = A0W_, KS = KS_;
  static constexpr bool HALF = HALF_;
  static constexpr int A0G = 8 * A0W / KS;
  static constexpr int RT = HALF ? 2 * NT - 1 : A0W * NT;
  static_assert(!HALF || A0W == 2, "HALF packs two values of a0");
};

// grid (ceil(n / A0G), nchunk), 512 threads (RhoShape; n padded to 16 NT with
// zeros).  MT: the element type the moments are read in (the FP32 form reads
// an FP32 copy, half the bytes of the staging loads that bound it).
//   What bounds it: FP64 (FP32) matrix cores.  Whole J, 16 values of a0 per
// work group in whole tiles against HALF with KS = 2, FP64: 500500 pairs at
// n = 40 3395 -> 2634 us (with the projection's HALF form), at n = 24 1090 ->
// 776 us.  FP32 keeps one value of a0 per wave: its packed form spilled (12
// orbitals at n = 40 799 -> 874 us), and splitting a batch would change the
// FP32 sums.
template <class Op, class Shape, class MT>
__device__ __forceinline__ void rho_mfma_body(const MT* __restrict__ M, const double* __restrict__ Dt, int n,
                                              int64_t npair, int64_t chunk, double* __restrict__ part) {
  constexpr int NT = Shape::NT, A0W = Shape::A0W, KS = Shape::KS, RT = Shape::RT;
  constexpr bool HALF = Shape::HALF;
  constexpr int NP = 16 * NT;                  // padded extent of a1 and a2
  constexpr int A0G = Shape::A0G;              // a0 per work group
  constexpr int ROWS = A0G + 2 * NP;           // staged rows: c (A0G), m1 (NP), m2 (NP)
  constexpr int PER = ROWS * kKB / 512;        // staged values per thread
  constexpr int CS = A0G + 1, MS = NP + 1;     // LDS row strides
  using T = typename Op::T;
  using Acc = typename Op::Acc;
  // two LDS buffers: batch b is read from buffer b & 1 while batch b + 1 is
  // stored into the other after the MFMAs, one barrier per batch
  constexpr int kBuf = kKB * (CS + 2 * MS);
  __shared__ __align__(16) T s_buf[2 * kBuf];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int a0base = blockIdx.x * A0G;
  const int wa = KS == 2 ? wave & 3 : wave, kh = KS == 2 ? wave >> 2 : 0;   // a0 values, share of the pairs
  const int64_t q0 = (int64_t)blockIdx.y * chunk;
  const int64_t q1 = (q0 + chunk < npair) ? q0 + chunk : npair;
  const MT* M0 = M;
  const MT* M1 = M + (int64_t)n * npair;
  const MT* M2 = M + 2 * (int64_t)n * npair;

  // staged value e = threadIdx.x + 512 i of a batch: row e / kKB, pair e % kKB
  T pre[PER];
  auto load = [&](int64_t qb) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 512 * i;
      const int row = e / kKB;
      const int64_t q = qb + (e % kKB);
      double v = 0.0;
      if (q < q1) {
        if (row < A0G) {
          const int a0 = a0base + row;
          if (a0 < n) v = Dt[q] * (double)M0[(int64_t)a0 * npair + q];
        } else if (row < A0G + NP) {
          const int a = row - A0G;
          if (a < n) v = (double)M1[(int64_t)a * npair + q];
        } else {
          const int a = row - A0G - NP;
          if (a < n) v = (double)M2[(int64_t)a * npair + q];
        }
      }
      pre[i] = (T)v;
    }
  };
  auto store = [&](T* buf) {
    T* s_m1 = buf + kKB * CS;
    T* s_m2 = s_m1 + kKB * MS;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 512 * i;
      const int row = e / kKB, qq = e % kKB;
      if (row < A0G) buf[qq * CS + row] = pre[i];
      else if (row < A0G + NP) s_m1[qq * MS + row - A0G] = pre[i];
      else s_m2[qq * MS + row - A0G - NP] = pre[i];
    }
  };
  // row block i of the wave: this lane's a0 (an offset) and a1
  auto row_a0 = [&](int i, int row) { return HALF ? (row >= n ? 1 : 0) : i / NT; };
  auto row_a1 = [&](int i, int row) { return HALF ? (row >= n ? row - n : row) : row - 16 * NT * (i / NT); };

  Acc acc[RT][NT];
  v4d tot[Op::kSplitSum ? RT : 1][NT];  // FP64 sums of the FP32 batches
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      acc[i][j] = Acc{0, 0, 0, 0};
      if constexpr (Op::kSplitSum) tot[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    }

  load(q0);
  store(s_buf);
  __syncthreads();
  int buf = 0;
  for (int64_t qb = q0; qb < q1; qb += kKB, buf ^= 1) {
    const bool more = qb + kKB < q1;
    if (more) load(qb + kKB);  // next batch in flight during the MFMAs
    const T* s_c = s_buf + buf * kBuf;
    const T* s_m1 = s_c + kKB * CS;
    const T* s_m2 = s_m1 + kKB * MS;
#pragma unroll(HALF && NT == 3 ? 1 : 2)   // more spills
    for (int st = 0; st < kKB / 4 / KS; ++st) {
      const int kk = 4 * (st + kh * (kKB / 4 / KS)) + kg;  // this lane's pair within the batch
      T bm[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) bm[j] = s_m2[kk * MS + 16 * j + r16];
      if constexpr (HALF) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const int row = 16 * i + r16;
          // rows past 2 n read the zeros staged for a1 >= n
          const T av = s_c[kk * CS + wa * A0W + row_a0(i, row)] * s_m1[kk * MS + row_a1(i, row)];
#pragma unroll
          for (int j = 0; j < NT; ++j) acc[i][j] = Op::mma(av, bm[j], acc[i][j]);
        }
      } else {
        T am[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) am[i] = s_m1[kk * MS + 16 * i + r16];
#pragma unroll
        for (int a = 0; a < A0W; ++a) {
          const T cq = s_c[kk * CS + wa * A0W + a];
#pragma unroll
          for (int i = 0; i < NT; ++i) {
            const T av = cq * am[i];
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[a * NT + i][j] = Op::mma(av, bm[j], acc[a * NT + i][j]);
          }
        }
      }
    }
    if constexpr (Op::kSplitSum) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
          for (int r = 0; r < 4; ++r) tot[i][j][r] += (double)acc[i][j][r];
          acc[i][j] = Acc{0, 0, 0, 0};
        }
    }
    // the other buffer was last read in the previous batch, which every wave
    // finished before the barrier that ended it
    if (more) store(s_buf + (buf ^ 1) * kBuf);
    __syncthreads();
  }
  auto sums = [&](int i, int j) -> v4d& {
    if constexpr (Op::kSplitSum) return tot[i][j];
    else return acc[i][j];
  };

  if constexpr (KS == 2) {
    // the upper waves' sums, as many row blocks at a time as the buffers hold
    constexpr int kFit = (int)(sizeof(T) * 2 * kBuf / (4 * NT * 64 * sizeof(v4d)));
    constexpr int FIT = kFit < RT ? kFit : RT;
    static_assert(FIT >= 1, "a row block of four waves fits in the buffers");
    v4d* s_sum = reinterpret_cast<v4d*>(s_buf);
#pragma unroll
    for (int i0 = 0; i0 < RT; i0 += FIT) {
      if (i0 > 0) __syncthreads();
      if (kh == 1) {
#pragma unroll
        for (int i = i0; i < i0 + FIT && i < RT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) s_sum[((wa * FIT + i - i0) * NT + j) * 64 + lane] = sums(i, j);
      }
      __syncthreads();
      if (kh == 0) {
#pragma unroll
        for (int i = i0; i < i0 + FIT && i < RT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j) sums(i, j) += s_sum[((wa * FIT + i - i0) * NT + j) * 64 + lane];
      }
    }
    if (kh == 1) return;
  }

  // lane l holds column a2 = 16 j + l%16 and packed rows 16 i + row_of(l/16, r)
  const int64_t n2 = (int64_t)n * n;
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * i + Op::row_of(kg, r);
      const int a0 = a0base + wa * A0W + row_a0(i, row), a1 = row_a1(i, row);
      if (a0 >= n || a1 >= n) continue;
      double* out = part + ((int64_t)blockIdx.y * n + a0) * n2 + (int64_t)a1 * n;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int a2 = 16 * j + r16;
        if (a2 < n) out[a2] = sums(i, j)[r];
      }
    }
}

template <class Op, class Shape, class MT>
__global__ void __launch_bounds__(512, 1)
rho_mfma_kernel(const MT* __restrict__ M, const double* __restrict__ Dt, int n, int64_t npair,
                int64_t chunk, double* __restrict__ part) {
  // batched densities (several orbitals in one launch): density z, its
  // partial grids after those of densities 0 .. z-1
  rho_mfma_body<Op, Shape, MT>(M, Dt + (int64_t)blockIdx.z * npair, n, npair, chunk,
                                 part + (int64_t)blockIdx.z * gridDim.y * n * n * n);
}

// Pair lists cut into consecutive spans (the partitions of the adaptive
// boxes): span z holds pairs off[z] .. off[z+1] of the list, its moments the
// block M + 3 n off[z] (each span's own pair count as the stride); blk[z] is
// the first work group of span z in a launch that covers all spans.
struct Spans {
  int64_t off[kMaxParts + 1];
  int64_t blk[kMaxParts + 1];
};

// rho of every span in one launch: grid (ceil(n / A0G), nchunk, nspan),
// span z's pairs cut into nchunk chunks, its partial grids after those of
// spans 0 .. z-1.  An empty span writes zero partial grids.
template <class Op, class Shape, class MT>
__global__ void __launch_bounds__(512, 1)
rho_spans_kernel(const MT* __restrict__ M, const double* __restrict__ Dt, int n, Spans sp, double* __restrict__ part) {
  const int z = blockIdx.z;
  const int64_t cnt = sp.off[z + 1] - sp.off[z];
  const int64_t chunk = (cnt + gridDim.y - 1) / gridDim.y;
  rho_mfma_body<Op, Shape, MT>(M + 3 * (int64_t)n * sp.off[z], Dt + sp.off[z], n, cnt, chunk,
                                 part + (int64_t)z * gridDim.y * n * n * n);
}

// ---------------------------------------------------------------------------
// Split-BF16 forms of the two pair contractions (TAI_BF16X3, TAI_BF16X6).
// Each FP32 operand value x is cut into S bfloat16 slices, s0 = bf16(x),
// s1 = bf16(x - s0), s2 = bf16(x - s0 - s1), and a product sums s_i t_j over
// i + j <= S - 1 on the matrix cores (v_mfma_f32_16x16x32_bf16, FP32
// accumulation): S = 2 gives 3 products, S = 3 gives 6.  bfloat16 keeps
// FP32's exponent range, so no operand scaling is needed.  The moments are
// read from the FP32 copy, the grid sums and mode products stay FP64.
//
// Measured on the device, sums on these MFMAs lose more than an exactly
// rounded FP32 accumulation would: J on the Nb = 64 workload was about 4x
// less accurate than a host model with round-to-nearest accumulation, close
// to one with truncating accumulation.  Each accumulator therefore takes few
// MFMA additions: in rho the small cross products of a K-step are summed in
// a fresh accumulator and folded into the running sum with one VALU add
// (round-to-nearest), and in J_p the 32-wide K-chunks go round-robin into
// three accumulators that are added the same way.  The pair sums of rho
// cancel heavily, and even so the 6-product rho stayed several times less
// accurate than the FP32 one (1.3e-6 against 1.9e-7 relative 2-norm of J
// on a 300-function basis), so TAI_BF16X6 takes the FP32 rho and splits
// only the projection; TAI_BF16X3 runs both contractions split.
// ---------------------------------------------------------------------------
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

template <int S>
__device__ inline void split8(const float (&x)[8], v8bf (&out)[S]) {
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = x[e];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const __bf16 h = (__bf16)r[e];
      out[s][e] = h;
      r[e] -= (float)h;
    }
}

__device__ inline v4f mma_bf16(v8bf a, v8bf b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// slice pairs (A slice, B slice) summed by an S-slice product
template <int S> struct SlicePairs;
template <> struct SlicePairs<2> {
  static constexpr int kN = 3;
  static constexpr int a[3] = {0, 0, 1};
  static constexpr int b[3] = {0, 1, 0};
};
template <> struct SlicePairs<3> {
  static constexpr int kN = 6;
  static constexpr int a[6] = {0, 0, 1, 0, 1, 2};
  static constexpr int b[6] = {0, 1, 0, 2, 1, 0};
};

constexpr int kKB16 = 64;   // pairs per LDS batch of the split rho kernel (two K-steps of 32)

// rho partials in split BF16.  1D grid; block b runs on XCD b % 8 and takes
// a0 group g and pair chunk c with the ngroups groups of one chunk on one XCD
// one after another, so that the chunk's moments are read from that XCD's L2
// by all its groups.  Wave w owns a0 = 8 A0W g + A0W w + {0 .. A0W-1} and all (a1, a2)
// in NT x NT tiles of 16 x 16; per batch of 64 pairs the chunk's rows
// c(a0, q) = Dt_q m_{q,0}(a0) (FP32), m_1 (FP32) and the slices of m_2 are
// staged in LDS, K-contiguous per row.  The A operand c(a0, q) m_{q,1}(a1) is
// formed in FP32 per lane and split on the fly.  Products are summed in FP32
// within one batch and in FP64 across the batches of the chunk; the chunk
// partials are summed in FP64 in a fixed order.
template <int NT, int S, int A0W>
__global__ void __launch_bounds__(512, 1)
rho16_kernel(const float* __restrict__ M, const double* __restrict__ Dt, int n, int64_t npair, int64_t chunk,
             int nchunk, int ngroups, double* __restrict__ part) {
  constexpr int NP = 16 * NT;
  constexpr int A0G = 8 * A0W;
  constexpr int CST = kKB16 + 4;          // FP32 row stride of s_c, s_m1 (floats)
  constexpr int BST = kKB16 + 8;          // bf16 row stride of the m_2 slices
  constexpr int ROWS = A0G + 2 * NP;      // staged rows per batch
  constexpr int PER = ROWS * kKB16 / 512; // staged values per thread
  using SP = SlicePairs<S>;
  __shared__ __align__(16) float s_c[2][A0G * CST];
  __shared__ __align__(16) float s_m1[2][NP * CST];
  __shared__ __align__(16) __bf16 s_m2[2][S * NP * BST];
  const int b = blockIdx.x;
  const int xcd = b & 7, r8 = b >> 3;
  const int g = r8 % ngroups;
  const int c = (r8 / ngroups) * 8 + xcd;
  if (c >= nchunk) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int a0base = g * A0G;
  const int64_t q0 = (int64_t)c * chunk;
  const int64_t q1 = (q0 + chunk < npair) ? q0 + chunk : npair;
  const float* M0 = M;
  const float* M1 = M + (int64_t)n * npair;
  const float* M2 = M + 2 * (int64_t)n * npair;
  // staged value e = threadIdx.x + 512 i: row e / 64, pair e % 64 (the pair
  // column is threadIdx.x % 64 for every i)
  const int qq = threadIdx.x & 63;
  float pre[PER];
  auto load = [&](int64_t qb) {
    const int64_t q = qb + qq;
    const bool ok = q < q1;
    const float dt = ok ? (float)Dt[q] : 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int row = (threadIdx.x + 512 * i) >> 6;
      float v = 0.f;
      if (ok) {
        if (row < A0G) {
          const int a0 = a0base + row;
          if (a0 < n) v = dt * M0[(int64_t)a0 * npair + q];
        } else if (row < A0G + NP) {
          const int a = row - A0G;
          if (a < n) v = M1[(int64_t)a * npair + q];
        } else {
          const int a = row - A0G - NP;
          if (a < n) v = M2[(int64_t)a * npair + q];
        }
      }
      pre[i] = v;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int row = (threadIdx.x + 512 * i) >> 6;
      if (row < A0G) s_c[buf][row * CST + qq] = pre[i];
      else if (row < A0G + NP) s_m1[buf][(row - A0G) * CST + qq] = pre[i];
      else {
        const int a = row - A0G - NP;
        float rr = pre[i];
#pragma unroll
        for (int sl = 0; sl < S; ++sl) {
          const __bf16 h = (__bf16)rr;
          s_m2[buf][(sl * NP + a) * BST + qq] = h;
          rr -= (float)h;
        }
      }
    }
  };

  v4f acc[A0W][NT][NT];
  v4d tot[A0W][NT][NT];
#pragma unroll
  for (int a = 0; a < A0W; ++a)
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        acc[a][i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        tot[a][i][j] = v4d{0.0, 0.0, 0.0, 0.0};
      }

  load(q0);
  store(0);
  __syncthreads();
  int buf = 0;
  for (int64_t qb = q0; qb < q1; qb += kKB16, buf ^= 1) {
    const bool more = qb + kKB16 < q1;
    if (more) load(qb + kKB16);
#pragma unroll
    for (int ks = 0; ks < kKB16 / 32; ++ks) {
      const int k0 = 32 * ks + 8 * kg;   // this lane's 8 pairs of the K-step
      v8bf bm[NT][S];
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int sl = 0; sl < S; ++sl)
          bm[j][sl] = *reinterpret_cast<const v8bf*>(&s_m2[buf][(sl * NP + 16 * j + r16) * BST + k0]);
      float cv[A0W][8];
#pragma unroll
      for (int a = 0; a < A0W; ++a) {
        const float4* src = reinterpret_cast<const float4*>(&s_c[buf][(A0W * wave + a) * CST + k0]);
        const float4 u = src[0], v = src[1];
        cv[a][0] = u.x; cv[a][1] = u.y; cv[a][2] = u.z; cv[a][3] = u.w;
        cv[a][4] = v.x; cv[a][5] = v.y; cv[a][6] = v.z; cv[a][7] = v.w;
      }
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const float4* src = reinterpret_cast<const float4*>(&s_m1[buf][(16 * i + r16) * CST + k0]);
        const float4 u = src[0], v = src[1];
        const float m1v[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
        for (int a = 0; a < A0W; ++a) {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = cv[a][e] * m1v[e];
          v8bf as[S];
          split8<S>(x, as);
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            // cross products of the slices in a fresh accumulator, the
            // leading product into the running sum, then one rounded add
            v4f lo = mma_bf16(as[SP::a[1]], bm[j][SP::b[1]], v4f{0.f, 0.f, 0.f, 0.f});
#pragma unroll
            for (int pp = 2; pp < SP::kN; ++pp) lo = mma_bf16(as[SP::a[pp]], bm[j][SP::b[pp]], lo);
            acc[a][i][j] = mma_bf16(as[0], bm[j][0], acc[a][i][j]);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][i][j][r] += lo[r];
          }
        }
      }
    }
#pragma unroll
    for (int a = 0; a < A0W; ++a)
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
          for (int r = 0; r < 4; ++r) tot[a][i][j][r] += (double)acc[a][i][j][r];
          acc[a][i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    if (more) store(buf ^ 1);
    __syncthreads();
  }
  // lane l holds column a2 = 16 j + l%16 and rows a1 = 16 i + 4 (l/16) + r
  const int64_t n2 = (int64_t)n * n;
#pragma unroll
  for (int a = 0; a < A0W; ++a) {
    const int a0 = a0base + A0W * wave + a;
    if (a0 >= n) continue;
    double* out = part + ((int64_t)c * n + a0) * n2;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a1 = 16 * i + 4 * kg + r, a2 = 16 * j + r16;
          if (a1 < n && a2 < n) out[a1 * n + a2] = tot[a][i][j][r];
        }
  }
}

// Part y of ny of the a0 values, cut at even values (the pairs of a0 values of
// the HALF form start at the same places in every split).
__device__ inline void a0_range(int n, int y, int ny, int& alo, int& ahi) {
  const int h = (n + 1) / 2;
  alo = min(n, 2 * (y * h / ny));
  ahi = min(n, 2 * ((y + 1) * h / ny));
}

// Inner layout of the split J_p contraction: position pos = nseg a2 + s
// (segment-minor) holds slice a[s] of Phi(.., a2) on the A side and slice
// b[s] of m_2(a2) on the B side, zero padded to kc = 32 ceil(nseg n / 32).
// Eight consecutive positions (one lane's share of a 32-wide K-step) then
// touch at most three values of a2 for nseg = 6.
template <int S> struct JSeg;
template <> struct JSeg<2> {
  static constexpr int kSeg = 3;
  static constexpr int a[3] = {0, 0, 1};
  static constexpr int b[3] = {0, 1, 0};
};
template <> struct JSeg<3> {
  static constexpr int kSeg = 6;
  static constexpr int a[6] = {0, 0, 1, 0, 1, 2};
  static constexpr int b[6] = {0, 1, 0, 2, 1, 0};
};
__host__ __device__ inline int j16_kc(int S, int n) {
  const int nseg = S == 2 ? 3 : 6;
  return (nseg * n + 31) / 32 * 32;
}

// Phi split into its slices in the A layout: Ps[a0][a1][kc] (bf16), for the
// grid tensors of one or several spans one after another.
template <int S>
__global__ void __launch_bounds__(256)
phi_split_kernel(const double* __restrict__ Phi, int n, int kc, __bf16* __restrict__ Ps) {
  const int64_t row = blockIdx.x;            // (a0, a1)
  const double* src = Phi + row * n;
  __bf16* dst = Ps + row * kc;
  constexpr int NS = JSeg<S>::kSeg;
  for (int pos = threadIdx.x; pos < kc; pos += 256) {
    const int a2 = pos / NS, seg = pos - a2 * NS;
    __bf16 v = (__bf16)0.f;
    if (a2 < n) {
      const int want = JSeg<S>::a[seg];
      double r = src[a2];
      for (int sl = 0; sl < want; ++sl) r -= (double)(float)(__bf16)(float)r;
      v = (__bf16)(float)r;
    }
    dst[pos] = v;
  }
}

// J_p in split BF16 for 256 pairs per work group of 512 threads (wave w owns
// the two 16-pair tiles at blk*256 + 32 w).  Each lane holds the m_2
// slices of its pair in the B layout for the whole kernel; per a0 the slab
// Ps(a0, :, :) is staged in LDS (double-buffered) and X = Phi(a0) m_2 comes
// out of the matrix cores one 16-row block of a1 at a time, contracted at
// once with m_1 (FP32) and, per a0, with m_0 (FP64).  All spans in one launch
// and the a0 values split over grid y, as in jp_spans_kernel: four boxes of
// 7844 pairs each (n = 40) kept 31 compute units busy four times over.
template <int NT, int S, int KC>
__global__ void __launch_bounds__(512, 1)
jp16_kernel(const float* __restrict__ Mall, const __bf16* __restrict__ Psall, int n, int nspan, Spans sp,
            double* __restrict__ Jpall, int64_t len) {
  int z = 0;
  while (z + 1 < nspan && (int64_t)blockIdx.x >= sp.blk[z + 1]) ++z;
  const int64_t off = sp.off[z], npair = sp.off[z + 1] - off, blk = (int64_t)blockIdx.x - sp.blk[z];
  const float* M = Mall + 3 * (int64_t)n * off;
  const __bf16* Ps = Psall + (int64_t)z * n * n * (32 * KC);
  double* Jp = Jpall + blockIdx.y * len + off;
  int alo, ahi;
  a0_range(n, blockIdx.y, gridDim.y, alo, ahi);
  constexpr int PT = 2;
  constexpr int kc = 32 * KC;
  constexpr int RS = kc + 8;                       // LDS row stride (bf16)
  constexpr int Q16 = kc / 8;                      // 16-byte pieces per row
  __shared__ __align__(16) __bf16 s_p[2][NT * 16 * RS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const float* M0 = M;
  const float* M1 = M + (int64_t)n * npair;
  const float* M2 = M + 2 * (int64_t)n * npair;
  const int64_t n2kc = (int64_t)n * kc;

  int64_t pc[PT];
  bool pok[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int64_t p = blk * 256 + wave * 32 + 16 * t + r16;
    pok[t] = p < npair;
    pc[t] = pok[t] ? p : 0;
  }
  // B fragments: K positions 32 c + 8 kg + e of the B layout; the lane's
  // eight positions hold the slices of at most NA consecutive values of a2.
  // One code path per kg, so that every position maps to its (a2, slice) at
  // compile time.
  constexpr int NS = JSeg<S>::kSeg;
  constexpr int NA = (7 + NS - 1) / NS + 1;
  v8bf bm[PT][KC];
  auto build_b = [&](auto kgc) {
    constexpr int KG = decltype(kgc)::value;
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
      for (int cc = 0; cc < KC; ++cc) {
        const int pos0 = 32 * cc + 8 * KG;
        const int a2f = pos0 / NS;
        float sl[NA][S];
#pragma unroll
        for (int u = 0; u < NA; ++u) {
          const int a2 = a2f + u;
          float r = (pok[t] && a2 < n) ? M2[(int64_t)a2 * npair + pc[t]] : 0.f;
#pragma unroll
          for (int q = 0; q < S; ++q) {
            const __bf16 h = (__bf16)r;
            sl[u][q] = (float)h;
            r -= (float)h;
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int pos = pos0 + e;
          bm[t][cc][e] = (__bf16)sl[pos / NS - a2f][JSeg<S>::b[pos % NS]];
        }
      }
  };
  switch (kg) {
    case 0: build_b(std::integral_constant<int, 0>{}); break;
    case 1: build_b(std::integral_constant<int, 1>{}); break;
    case 2: build_b(std::integral_constant<int, 2>{}); break;
    default: build_b(std::integral_constant<int, 3>{}); break;
  }
  // m_1 at this lane's output rows a1 = 16 i + 4 kg + r
  float w1[PT][NT][4];
#pragma unroll
  for (int t = 0; t < PT; ++t)
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a1 = 16 * i + 4 * kg + r;
        w1[t][i][r] = (pok[t] && a1 < n) ? M1[(int64_t)a1 * npair + pc[t]] : 0.f;
      }

  // slab staging: rows a1 < 16 NT (zero beyond n), Q16 pieces of 16 bytes each
  constexpr int PIECES = NT * 16 * Q16;
  constexpr int PER = (PIECES + 511) / 512;
  uint4 pre[PER];
  auto load = [&](int a0) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 512 * i;
      const int a1 = e / Q16, q = e - a1 * Q16;
      uint4 v = uint4{0u, 0u, 0u, 0u};
      if (e < PIECES && a1 < n) v = reinterpret_cast<const uint4*>(Ps + a0 * n2kc + (int64_t)a1 * kc)[q];
      pre[i] = v;
    }
  };
  auto store = [&](__bf16* bufp) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 512 * i;
      if (e < PIECES) {
        const int a1 = e / Q16, q = e - a1 * Q16;
        *reinterpret_cast<uint4*>(bufp + a1 * RS + 8 * q) = pre[i];
      }
    }
  };

  double jacc[PT] = {};
  if (alo < ahi) load(alo);
  for (int a0 = alo; a0 < ahi; ++a0) {
    __bf16* bufp = s_p[a0 & 1];
    store(bufp);
    __syncthreads();  // slab a0 in LDS; every wave is past slab a0-2 in this buffer
    if (a0 + 1 < ahi) load(a0 + 1);
    double y[PT] = {};
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      // the K-chunks go round-robin into NR accumulators (at most three
      // MFMA additions each), summed with rounded adds at the end
      constexpr int NR = KC < 3 ? KC : 3;
      v4f Xr[NR][PT];
#pragma unroll
      for (int u = 0; u < NR; ++u)
#pragma unroll
        for (int t = 0; t < PT; ++t) Xr[u][t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int cc = 0; cc < KC; ++cc) {
        const v8bf av = *reinterpret_cast<const v8bf*>(bufp + (16 * i + r16) * RS + 32 * cc + 8 * kg);
#pragma unroll
        for (int t = 0; t < PT; ++t) Xr[cc % NR][t] = mma_bf16(av, bm[t][cc], Xr[cc % NR][t]);
      }
      v4f X[PT];
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        X[t] = Xr[0][t];
#pragma unroll
        for (int u = 1; u < NR; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) X[t][r] += Xr[u][t][r];
      }
#pragma unroll
      for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) y[t] += (double)w1[t][i][r] * (double)X[t][r];
    }
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      const double m0 = pok[t] ? (double)M0[(int64_t)a0 * npair + pc[t]] : 0.0;
      jacc[t] += m0 * y[t];
    }
  }
  // the four lanes l/16 = 0..3 of a column hold partial sums over a1
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    double v = jacc[t];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (kg == 0 && pok[t]) Jp[pc[t]] = v;
  }
}

// J_p for 256 pairs per work group of 512 threads: wave w owns the two
// 16-pair tiles at blk*256 + 32 w.  The rows (a0, a1) of Phi are taken A0P
// values of a0 at a time: the slab Phi(a0 .. a0 + A0P - 1, :, :) is staged in
// LDS (double-buffered, the next slab's loads in flight during the MFMAs);
// X = Phi(a0 ..) m_2 comes out of the matrix cores one block of 16 rows at a
// time and is contracted at once with m_1 and m_0.
//   HALF: n <= 16 NT - 8.  Two values of a0 then fill 2 NT - 1 blocks of rows
// instead of 2 NT, and the inner index stops at 16 NT - 8: at n = 40, 50 MFMAs
// per pair of a0 values instead of 72, at n = 24 18 instead of 32.  Otherwise
// one value of a0 per slab, whose weights m_1 take half the registers.
//   a0 in [alo, ahi): the launch splits the a0 values where the pairs alone
// leave the chip idle (jp_splits), each part writing its own sums.
template <class Op, int NT, bool HALF>
__device__ __forceinline__ void jp_mfma_body(const double* __restrict__ M, const double* __restrict__ Phi, int n,
                                             int64_t npair, double* __restrict__ Jp, int64_t blk, int alo, int ahi) {
  constexpr int A0P = HALF ? 2 : 1, RT = HALF ? 2 * NT - 1 : NT, NK = HALF ? 4 * NT - 2 : 4 * NT, PT = 2;
  constexpr int ROWS = 16 * RT, COLS = 4 * NK;
  constexpr int PS = COLS + 1;                      // LDS row stride
  constexpr int SLAB = ROWS * COLS;                 // padded slab values
  constexpr int PER = (SLAB + 511) / 512;           // staged values per thread
  using T = typename Op::T;
  using Acc = typename Op::Acc;
  __shared__ T s_phi[2][ROWS * PS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const double* M0 = M;
  const double* M1 = M + (int64_t)n * npair;
  const double* M2 = M + 2 * (int64_t)n * npair;
  const int64_t n2 = (int64_t)n * n;

  int64_t pc[PT];
  bool pok[PT];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    const int64_t p = blk * 256 + wave * 32 + 16 * t + r16;
    pok[t] = p < npair;
    pc[t] = pok[t] ? p : 0;
  }
  // B fragments m_2(a2 = 4 s + l/16, p) and the weights m_1(a1, p) of this
  // lane's output rows (a0 offset, a1), offset n + a1 = 16 i + row_of(l/16, r)
  T bm[PT][NK];
  double w1[PT][RT][4];
#pragma unroll
  for (int t = 0; t < PT; ++t) {
#pragma unroll
    for (int st = 0; st < NK; ++st) {
      const int a2 = 4 * st + kg;
      bm[t][st] = (T)((pok[t] && a2 < n) ? M2[(int64_t)a2 * npair + pc[t]] : 0.0);
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + Op::row_of(kg, r);
        const int a1 = HALF && row >= n ? row - n : row;
        w1[t][i][r] = (pok[t] && a1 < n) ? M1[(int64_t)a1 * npair + pc[t]] : 0.0;
      }
  }

  double pre[PER];
  auto load = [&](int a0) {
    const int rows = min(A0P, ahi - a0) * n;        // rows past the a0 range are zero
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 512 * i;
      const int row = e / COLS, a2 = e % COLS;
      pre[i] = (e < SLAB && row < rows && a2 < n) ? Phi[a0 * n2 + (int64_t)row * n + a2] : 0.0;
    }
  };
  auto store = [&](T* buf) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 512 * i;
      if (e < SLAB) buf[(e / COLS) * PS + (e % COLS)] = (T)pre[i];
    }
  };

  double jacc[PT] = {};
  if (alo < ahi) load(alo);
  int par = 0;
  for (int a0 = alo; a0 < ahi; a0 += A0P, par ^= 1) {
    T* buf = s_phi[par];
    store(buf);
    __syncthreads();  // this slab in LDS; every wave is past the slab before the last in this buffer
    if (a0 + A0P < ahi) load(a0 + A0P);
    double m0v[A0P][PT];
#pragma unroll
    for (int u = 0; u < A0P; ++u)
#pragma unroll
      for (int t = 0; t < PT; ++t)
        m0v[u][t] = (pok[t] && a0 + u < ahi) ? M0[(int64_t)(a0 + u) * npair + pc[t]] : 0.0;
    double y[A0P][PT] = {};
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      Acc X[PT];
#pragma unroll
      for (int t = 0; t < PT; ++t) X[t] = Acc{0, 0, 0, 0};
#pragma unroll
      for (int st = 0; st < NK; ++st) {
        const T av = buf[(16 * i + r16) * PS + 4 * st + kg];
#pragma unroll
        for (int t = 0; t < PT; ++t) X[t] = Op::mma(av, bm[t][st], X[t]);
      }
      // the block's rows belong to one value of a0, or the block holds the
      // boundary between the two
      if (!HALF || 16 * i + 15 < n) {
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) y[0][t] += w1[t][i][r] * (double)X[t][r];
      } else if (16 * i >= n) {
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) y[A0P - 1][t] += w1[t][i][r] * (double)X[t][r];
      } else {
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const bool first = 16 * i + Op::row_of(kg, r) < n;
            const double v = w1[t][i][r] * (double)X[t][r];
            y[0][t] += first ? v : 0.0;
            y[A0P - 1][t] += first ? 0.0 : v;
          }
      }
    }
#pragma unroll
    for (int u = 0; u < A0P; ++u)
#pragma unroll
      for (int t = 0; t < PT; ++t) jacc[t] += m0v[u][t] * y[u][t];
  }
  // the four lanes l/16 = 0..3 of a column hold partial sums over a1
#pragma unroll
  for (int t = 0; t < PT; ++t) {
    double v = jacc[t];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (kg == 0 && pok[t]) Jp[pc[t]] = v;
  }
}

// J_p of every span in one launch: work groups blk[z] .. blk[z+1] take the
// pairs of span z (256 each) against its own Phi (Phi + z n^3); one span is the
// plain J.  Grid y splits the a0 values; part y's sums go to Jp + y len.
template <class Op, int NT, bool HALF>
__global__ void __launch_bounds__(512, 1)
jp_spans_kernel(const double* __restrict__ M, const double* __restrict__ Phi, int n, int nspan, Spans sp,
                double* __restrict__ Jp, int64_t len) {
  int z = 0;
  while (z + 1 < nspan && (int64_t)blockIdx.x >= sp.blk[z + 1]) ++z;
  const int64_t o = sp.off[z];
  int alo, ahi;
  a0_range(n, blockIdx.y, gridDim.y, alo, ahi);
  jp_mfma_body<Op, NT, HALF>(M + 3 * (int64_t)n * o, Phi + (int64_t)z * n * n * n, n, sp.off[z + 1] - o,
                             Jp + blockIdx.y * len + o, (int64_t)blockIdx.x - sp.blk[z], alo, ahi);
}

// J from the sums over the a0 values of the J_p launch: parts 0 .. nsplit - 1
// in order, part y at Jp + y npair.
__global__ void __launch_bounds__(256)
unpack_kernel(const double* __restrict__ Jp, int nsplit, int nb, int64_t npair, const int32_t* __restrict__ pairs,
              double* __restrict__ J) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npair) return;
  int mu, nu;
  if (!pair_of(pairs, nb, p, mu, nu)) return;
  double v = Jp[p];
  for (int y = 1; y < nsplit; ++y) v += Jp[y * npair + p];
  J[(int64_t)mu * nb + nu] = v;
  J[(int64_t)nu * nb + mu] = v;
}

// Pair density of one orbital, D = q q^T folded over the ordered pairs:
// Dt_p = q(mu) q(nu) (2 - delta_mu,nu).
__global__ void __launch_bounds__(256)
orbital_pairs_kernel(const double* __restrict__ q, int nb, int64_t npair, const int32_t* __restrict__ pairs,
                     double* __restrict__ Dt) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npair) return;
  q += (int64_t)blockIdx.y * nb;   // orbital blockIdx.y
  Dt += (int64_t)blockIdx.y * npair;
  int mu, nu;
  Dt[p] = pair_of(pairs, nb, p, mu, nu) ? q[mu] * q[nu] * (mu == nu ? 1.0 : 2.0) : 0.0;
}

// J_mo(i, j) = sum_a rho_i(a) Phi_j(a) over the n^3 grid, one work group per
// (i, j), a fixed-order tree sum.
__global__ void __launch_bounds__(256)
mo_dot_kernel(const double* __restrict__ R, const double* __restrict__ F, int64_t n3, int norb, double scale,
              double* __restrict__ Jmo) {
  __shared__ double red[256];
  const int i = blockIdx.y, j = blockIdx.x;
  const double* r = R + (int64_t)i * n3;
  const double* f = F + (int64_t)j * n3;
  double acc = 0.0;
  for (int64_t a = threadIdx.x; a < n3; a += 256) acc += r[a] * f[a];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) Jmo[(int64_t)i * norb + j] = scale * red[0];
}

// J entries of the pairs that screening dropped are zero.
__global__ void __launch_bounds__(256) zero_kernel(double* __restrict__ x, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) x[i] = 0.0;
}

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }
inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

namespace {
// a0 groups the chunk capacity of the rho partials is counted with
int rho_groups(int prec, int n) {
  const int per = prec == kFP64 && n <= 48 ? 16 : 8;
  return (n + per - 1) / per;
}
// n fits 16 NT - 8 for its number of tiles NT <= 3
bool half_tiles(int n) { return n <= 48 && (n + 15) / 16 * 16 - n >= 8; }
// Values of a0 per work group of the shape that rho takes (with_rho_shape)
// for `chunks` chunks over all pair lists.  FP64 up to n = 48 with whole tiles:
// 16, or 8 (KS = 2) where 16 would leave half the compute units without a work
// group; measured, whole J at n = 32 in us: 38 work groups of 16 90, of 8 74;
// 146 either way 131; 226 120 and 124; n = 48, 237 236 and 246.
int rho_a0_group(int prec, int n, int64_t chunks) {
  return prec == kFP64 && n <= 48 && !half_tiles(n) && (int64_t)((n + 15) / 16) * chunks >= 128 ? 16 : 8;
}
}  // namespace

int j_nchunk(int prec, int n, int npair) {
  int c = kRhoGroups / rho_groups(prec, n);
  if (c < 1) c = 1;
  const int maxc = (npair + 4 * kKB - 1) / (4 * kKB);  // at least four batches per chunk
  if (c > maxc) c = maxc;
  return c < 1 ? 1 : c;
}

// the split-BF16 forms of J, TAI_BF16X3 (2 slices) and TAI_BF16X6 (3)
inline bool split_j(int prec) { return prec == kBF16X3 || prec == kBF16X6; }
inline int j_slices(int prec) { return prec == kBF16X6 ? 3 : 2; }

size_t j_work_bytes(int prec, int nq, int n, int npair) {
  const size_t n3 = (size_t)n * n * n;
  const int nc = j_nchunk(prec, n, npair);
  const size_t m32 = (prec == kFP32 || split_j(prec)) ? align256(4 * 3 * (size_t)n * npair) : 0;
  const size_t ps = split_j(prec) ? align256(2 * (size_t)n * n * j16_kc(j_slices(prec), n)) : 0;
  return align256(8 * (size_t)npair) * 2 + align256(8 * n3 * nc) + align256(8 * n3) * 2 + align256(8 * n3 * nq) * 2 +
         align256(8 * (size_t)nq) + m32 + ps;
}

JWork carve_j_work(void* base, int prec, int nq, int n, int npair) {
  const size_t n3 = (size_t)n * n * n;
  JWork w;
  w.nchunk = j_nchunk(prec, n, npair);
  char* p = static_cast<char*>(base);
  w.Dt = reinterpret_cast<double*>(p); p += align256(8 * (size_t)npair);
  w.Jp = reinterpret_cast<double*>(p); p += align256(8 * (size_t)npair);
  w.rho_part = reinterpret_cast<double*>(p); p += align256(8 * n3 * w.nchunk);
  w.rho = reinterpret_cast<double*>(p); p += align256(8 * n3);
  w.Phi = reinterpret_cast<double*>(p); p += align256(8 * n3);
  w.T1 = reinterpret_cast<double*>(p); p += align256(8 * n3 * nq);
  w.T2 = reinterpret_cast<double*>(p); p += align256(8 * n3 * nq);
  w.wsc = reinterpret_cast<double*>(p); p += align256(8 * (size_t)nq);
  w.M32 = (prec == kFP32 || split_j(prec)) ? reinterpret_cast<float*>(p) : nullptr;
  if (w.M32) p += align256(4 * 3 * (size_t)n * npair);
  w.Ps = split_j(prec) ? reinterpret_cast<void*>(p) : nullptr;
  return w;
}

namespace {
// Calls f with the shape of the rho kernel for n and a0 values per work group.
template <class Op, class F>
void with_rho_shape(int n, int a0g, F f) {
  auto shape = [&](auto nt) {
    constexpr int NT = decltype(nt)::value;
    if constexpr (NT == 4 || Op::kSplitSum) {
      f(RhoShape<NT, 1, false, 1>{});
    } else {
      if (half_tiles(n)) f(RhoShape<NT, 2, true, 2>{});
      else if (a0g == 16) f(RhoShape<NT, 2, false, 1>{});
      else f(RhoShape<NT, 2, false, 2>{});
    }
  };
  if (n <= 16) shape(std::integral_constant<int, 1>{});
  else if (n <= 32) shape(std::integral_constant<int, 2>{});
  else if (n <= 48) shape(std::integral_constant<int, 3>{});
  else shape(std::integral_constant<int, 4>{});
}

// Chunks of pairs a launch over nspan lists takes out of the capacity: what
// fills the target number of work groups.
int rho_chunks(int prec, int n, int nchunk, int nspan) {
  const int cap = nchunk / nspan;
  const int g = (n + 7) / 8;
  return half_tiles(n) && prec == kFP64 && cap > 1 ? std::max(1, std::min(cap, kRhoGroups / (g * nspan))) : cap;
}

// rho of ndens densities over one pair list into nchunk partial grids each
template <class Op, class MT>
void launch_pair_contraction_rho(int prec, const MT* M, int n, int npair, int nchunk, const double* Dt, double* part,
                                 hipStream_t s, int ndens = 1) {
  const int64_t chunk = ((int64_t)npair + nchunk - 1) / nchunk;
  const int a0g = rho_a0_group(prec, n, (int64_t)nchunk * ndens);
  const dim3 rg((n + a0g - 1) / a0g, nchunk, ndens);
  with_rho_shape<Op>(n, a0g, [&](auto sh) {
    hipLaunchKernelGGL((rho_mfma_kernel<Op, decltype(sh), MT>), rg, dim3(512), 0, s, M, Dt, n, (int64_t)npair, chunk,
                       part);
  });
}
}  // namespace

__global__ void __launch_bounds__(256) to_fp32_kernel(const double* __restrict__ x, int64_t count, float* __restrict__ y) {
  const int64_t i = grid_block() * blockDim.x + threadIdx.x;
  if (i < count) y[i] = (float)x[i];
}

namespace {
// Parts the a0 values of a J_p launch over `blocks` work groups are split
// into: least of rounds over the compute units times a work group's length, its
// a0 values plus a start (loading the pairs' moments) worth kJpStart of them.
// A second work group on a unit shares its matrix cores, so a round is one per
// unit.  Measured, whole J at n = 40 in us: 79 work groups 280 / 197 / 210 in
// 1 / 3 / 6 parts (FP64), 218 / 167 / 183 (FP32); 201 work groups, FP32, 279 in
// one part, 295 in five; 19 work groups at n = 32 147 in one part, 90 in
// eight; 240 or more: one.  room: how many parts' sums the caller can hold.
constexpr double kJpStart = 4.0;
int jp_splits(int64_t blocks, int n, int64_t room) {
  int best = 1;
  double best_t = 1e300;
  for (int y = 1; y <= 16 && y <= (n + 1) / 2 && y <= room; ++y) {
    const double t = (double)((blocks * y + 255) / 256) * ((double)n / y + kJpStart);
    if (t < best_t * (1.0 - 1e-9)) {
      best_t = t;
      best = y;
    }
  }
  return best;
}

// The spans of a J_p launch and where its sums go: one part straight into
// the pair vector, several into the partial grids of rho (free by then).
struct JpPlan {
  Spans sp{};
  int nspan = 1, splits = 1;
  int64_t total = 0;
  double* out = nullptr;
};
JpPlan jp_plan(const int64_t* offs, int nspan, int n, const JWork& w) {
  JpPlan p;
  p.nspan = nspan;
  p.total = offs[nspan];
  for (int z = 0; z <= nspan; ++z) {
    p.sp.off[z] = offs[z];
    p.sp.blk[z] = z == 0 ? 0 : p.sp.blk[z - 1] + nblk(offs[z] - offs[z - 1], 256);
  }
  const int64_t room = (int64_t)w.nchunk * n * n * n / (p.total > 0 ? p.total : 1);
  p.splits = jp_splits(p.sp.blk[nspan], n, room);
  p.out = p.splits > 1 ? w.rho_part : w.Jp;
  return p;
}

// J_p of the spans in FP64 or FP32 and J from it.
template <class Op>
void launch_jp(const double* M, int n, const int64_t* offs, int nspan, const double* Phi, const int32_t* pairs, int nb,
               const JWork& w, double* J, hipStream_t s) {
  const JpPlan p = jp_plan(offs, nspan, n, w);
  const dim3 g((unsigned)p.sp.blk[nspan], p.splits);
  auto go = [&](auto nt) {
    constexpr int NT = decltype(nt)::value;
    // beyond n = 48 the weights of two a0 values spill
    if (NT < 4 && n <= 16 * NT - 8)
      hipLaunchKernelGGL((jp_spans_kernel<Op, NT, (NT < 4)>), g, dim3(512), 0, s, M, Phi, n, nspan, p.sp, p.out,
                         p.total);
    else
      hipLaunchKernelGGL((jp_spans_kernel<Op, NT, false>), g, dim3(512), 0, s, M, Phi, n, nspan, p.sp, p.out, p.total);
  };
  if (n <= 16) go(std::integral_constant<int, 1>{});
  else if (n <= 32) go(std::integral_constant<int, 2>{});
  else if (n <= 48) go(std::integral_constant<int, 3>{});
  else go(std::integral_constant<int, 4>{});
  hipLaunchKernelGGL(unpack_kernel, dim3(nblk(p.total, 256)), dim3(256), 0, s, p.out, p.splits, nb, p.total, pairs, J);
}
}  // namespace

namespace {
template <int NT, int S>
void launch_rho16_t(const float* M, int n, int npair, const JWork& w, hipStream_t s) {
  constexpr int A0W = 1;   // one a0 per wave: FP32 and FP64 accumulators for 16 NT^2 outputs
  const int ng = (n + 8 * A0W - 1) / (8 * A0W);
  const int64_t chunk = ((int64_t)npair + w.nchunk - 1) / w.nchunk;
  const unsigned blocks = (unsigned)((w.nchunk + 7) / 8 * 8 * ng);
  hipLaunchKernelGGL((rho16_kernel<NT, S, A0W>), dim3(blocks), dim3(512), 0, s, M, w.Dt, n, (int64_t)npair, chunk,
                     w.nchunk, ng, w.rho_part);
}
template <int S>
void launch_rho16_s(const float* M, int n, int npair, const JWork& w, hipStream_t s) {
  if (n <= 16) launch_rho16_t<1, S>(M, n, npair, w, s);
  else if (n <= 32) launch_rho16_t<2, S>(M, n, npair, w, s);
  else if (n <= 48) launch_rho16_t<3, S>(M, n, npair, w, s);
  else launch_rho16_t<4, S>(M, n, npair, w, s);
}
// rho in split BF16 for TAI_BF16X3 only: TAI_BF16X6 takes the FP32 rho (the
// bf16 matrix cores' accumulation of the pair sums, which cancel heavily,
// left the 6-product rho several times less accurate than the FP32 one:
// 1.3e-6 against 1.9e-7 relative 2-norm of J on a 300-function basis)
void launch_rho16(int prec, const float* M, int n, int npair, const JWork& w, hipStream_t s) {
  (void)prec;
  launch_rho16_s<2>(M, n, npair, w, s);
}
inline bool rho_split(int prec) { return prec == kBF16X3; }

// J_p of the spans in split BF16 and J from it: every span's Phi cut into its
// slices (Ps: one span's slices, or room for all of them), then the
// contraction; the inner length kc (a multiple of 32) selects the compiled
// variant.
template <int S>
void launch_jp16(const float* M, int n, const int64_t* offs, int nspan, const double* Phi, void* Psv,
                 const int32_t* pairs, int nb, const JWork& w, double* J, hipStream_t s) {
  const int kc = j16_kc(S, n);
  __bf16* Ps = static_cast<__bf16*>(Psv);
  hipLaunchKernelGGL((phi_split_kernel<S>), dim3(nspan * n * n), dim3(256), 0, s, Phi, n, kc, Ps);
  const JpPlan p = jp_plan(offs, nspan, n, w);
  const dim3 g((unsigned)p.sp.blk[nspan], p.splits);
  const int NT = (n + 15) / 16, KC = kc / 32;
#define TAI_JP16(nt, kcc)                                                                                              \
  if (NT == nt && KC == kcc)                                                                                           \
  hipLaunchKernelGGL((jp16_kernel<nt, S, kcc>), g, dim3(512), 0, s, M, Ps, n, nspan, p.sp, p.out, p.total)
  if constexpr (S == 2) {
    // 3 n rounded up to 32: n <= 16 -> KC <= 2; <= 32 -> <= 3; <= 48 -> <= 5; <= 64 -> <= 6
    TAI_JP16(1, 1); TAI_JP16(1, 2);
    TAI_JP16(2, 2); TAI_JP16(2, 3);
    TAI_JP16(3, 4); TAI_JP16(3, 5);
    TAI_JP16(4, 5); TAI_JP16(4, 6);
  } else {
    // 6 n rounded up to 32: n <= 16 -> KC <= 3; <= 32 -> <= 6; <= 48 -> <= 9; <= 64 -> <= 12
    TAI_JP16(1, 1); TAI_JP16(1, 2); TAI_JP16(1, 3);
    TAI_JP16(2, 4); TAI_JP16(2, 5); TAI_JP16(2, 6);
    TAI_JP16(3, 7); TAI_JP16(3, 8); TAI_JP16(3, 9);
    TAI_JP16(4, 10); TAI_JP16(4, 11); TAI_JP16(4, 12);
  }
#undef TAI_JP16
  hipLaunchKernelGGL(unpack_kernel, dim3(nblk(p.total, 256)), dim3(256), 0, s, p.out, p.splits, nb, p.total, pairs, J);
}

// the FP32 pair contraction reads an FP32 copy of the moments (in w.M32),
// made once per call
void convert_moments(int prec, const double* M, int n, int npair, const JWork& w, hipStream_t s) {
  if (prec != kFP32 && !split_j(prec)) return;
  const int64_t count = 3 * (int64_t)n * npair;
  hipLaunchKernelGGL(to_fp32_kernel, grid_rows((count + 255) / 256), dim3(256), 0, s, M, count, w.M32);
}

// Phi = sum_k wsc_k rho x_0 K_k x_1 K_k x_2 K_k (wsc = (2/sqrt(pi)) w) on the
// FP64 matrix cores: the slab products into w.T1, the mode-0 products and
// node sum with the node runs' partial tensors in w.T2.  The plain J and the
// one-box adaptive J both take this exact sequence.
hipError_t launch_phi_grid(const double* rho, const double* K, const double* wsc, int n, int nq, const JWork& w,
                           double* Phi, hipStream_t s) {
  const int64_t n3 = (int64_t)n * n * n;
  return launch_mode_products(rho, 1, 1, K, 0, wsc, n, nq, w.T1, 1, 0, nq, Phi, w.T2, (int64_t)nq * n3, s);
}

// rho of one pair list from its pair densities Dt, in parity form on request
void launch_rho_list(int prec, const double* M, const float* M32, int n, int npair, const JWork& w, const double* Dt,
                     bool parity, double* rho, hipStream_t s) {
  int nchunk = w.nchunk;
  if (rho_split(prec)) {
    JWork wd = w;
    wd.Dt = const_cast<double*>(Dt);
    launch_rho16(prec, M32, n, npair, wd, s);
  } else {
    nchunk = rho_chunks(prec, n, nchunk, 1);
    if (prec == kFP64) launch_pair_contraction_rho<JF64>(prec, M, n, npair, nchunk, Dt, w.rho_part, s);
    else launch_pair_contraction_rho<JF32>(prec, M32, n, npair, nchunk, Dt, w.rho_part, s);
  }
  const int64_t n3 = (int64_t)n * n * n;
  if (parity) launch_parity_sum(w.rho_part, nchunk, 0, n3, n, 1, rho, s);
  else launch_sum_parts(w.rho_part, nchunk, n3, 1, rho, s);
}

// rho from the pair densities in w.Dt, then Phi = sum_k wsc_k rho x_d K_k (into
// w.rho and w.Phi), with the scaled weights in w.wsc
hipError_t launch_rho_phi(int prec, const double* M, int npair, int n, int nq, const NodeTables& tb, const JWork& w,
                          hipStream_t s) {
  launch_rho_list(prec, M, w.M32, n, npair, w, w.Dt, false, w.rho, s);
  return launch_phi_grid(w.rho, tb.K, w.wsc, n, nq, w, w.Phi, s);
}
// J_p and J of the spans in the arithmetic prec
void launch_projection(int prec, const double* M, const float* M32, int n, const int64_t* offs, int nspan,
                       const double* Phi, void* Ps, const int32_t* pairs, int nb, const JWork& w, double* J,
                       hipStream_t s) {
  if (prec == kBF16X6) launch_jp16<3>(M32, n, offs, nspan, Phi, Ps, pairs, nb, w, J, s);
  else if (prec == kBF16X3) launch_jp16<2>(M32, n, offs, nspan, Phi, Ps, pairs, nb, w, J, s);
  else if (prec == kFP32) launch_jp<JF32>(M, n, offs, nspan, Phi, pairs, nb, w, J, s);
  else launch_jp<JF64>(M, n, offs, nspan, Phi, pairs, nb, w, J, s);
}
}  // namespace

hipError_t launch_apply_j(int prec, const double* M, int nb, int npair, const int32_t* pairs, int n, int nq,
                          const NodeTables& tb, const double* D, double* J, const JWork& w, hipStream_t s) {
  hipLaunchKernelGGL(density_pairs_kernel, dim3(nblk(npair, 256)), dim3(256), 0, s, D, nb, (int64_t)npair, pairs,
                     w.Dt, ScaledWeights{tb.w, nq, 1, kTwoOverSqrtPi, w.wsc});
  convert_moments(prec, M, n, npair, w, s);
  const hipError_t e = launch_rho_phi(prec, M, npair, n, nq, tb, w, s);
  if (e != hipSuccess) return e;
  const int64_t whole[2] = {0, npair};
  if (pairs) {
    const int64_t nn = (int64_t)nb * nb;
    hipLaunchKernelGGL(zero_kernel, dim3(nblk(nn, 256)), dim3(256), 0, s, J, nn);
  }
  launch_projection(prec, M, w.M32, n, whole, 1, w.Phi, w.Ps, pairs, nb, w, J, s);
  return hipGetLastError();
}


// J over adaptive boxes (section 6.2 with eq. coulapprox): rho_s of every
// partition on its own grid, then for every partition s
//   Phi_s = (2/sqrt(pi)) sum_s' sum_k w_k rho_s' x_d K_k^(s,s')
// (the slab and mode-0 passes of each partition pair write their node
// products side by side, one weighted sum over the (s', k) blocks follows),
// J_p for the pairs of s, unpacked into J.
//
// One box runs the plain path's kernels (the same bits as tai_apply_J).
// More boxes: rho of all partitions in one launch (the single list's chunk
// count shared out among them), the mode products of all box pairs at once
// on the matrix cores with 2/sqrt(pi) folded into the repeated weights, and
// J_p of all partitions in one launch; the split-BF16 rho keeps a launch per
// partition.
namespace {
template <class Op, class MT>
void launch_rho_spans(int prec, const MT* M, int n, const Spans& sp, int nspan, int nchunk, const double* Dt,
                      double* part, hipStream_t s) {
  const int a0g = rho_a0_group(prec, n, (int64_t)nchunk * nspan);
  const dim3 rg((n + a0g - 1) / a0g, nchunk, nspan);
  with_rho_shape<Op>(n, a0g, [&](auto sh) {
    hipLaunchKernelGGL((rho_spans_kernel<Op, decltype(sh), MT>), rg, dim3(512), 0, s, M, Dt, n, sp, part);
  });
}
}  // namespace

hipError_t launch_apply_j_parts(int prec, const double* M, int nb, const int32_t* pairs, const int64_t* offs,
                                int nparts, int n, int nq, const double* w, double* Kx, const double* D,
                                double* J, const JWork& wk, double* rho_all, double* T2_all, double* Phi_all,
                                double* wrep, hipStream_t s) {
  const int64_t total = offs[nparts];
  const int64_t n3 = (int64_t)n * n * n, n2 = (int64_t)n * n;
  hipLaunchKernelGGL(density_pairs_kernel, dim3(nblk(total, 256)), dim3(256), 0, s, D, nb, total, pairs, wk.Dt,
                     ScaledWeights{w, nq, nparts, kTwoOverSqrtPi, wrep});
  convert_moments(prec, M, n, (int)total, wk, s);
  // one box: the plain path's sequence (the same bits as tai_apply_J); the
  // weights carry 2/sqrt(pi) either way
  const bool one = nparts == 1;
  const bool parity = !one && phi_octants(n, (int64_t)nparts * nparts);
  Spans sp{};
  for (int p = 0; p <= nparts; ++p) sp.off[p] = offs[p];
  // chunks per partition: the single list's count shared out, so that the
  // partial grids of all partitions fit where the list's would
  const int pchunk = wk.nchunk / nparts;
  if (!one && !rho_split(prec) && pchunk >= 1) {
    const int nchunk = rho_chunks(prec, n, wk.nchunk, nparts);
    if (prec == kFP64) launch_rho_spans<JF64>(prec, M, n, sp, nparts, nchunk, wk.Dt, wk.rho_part, s);
    else launch_rho_spans<JF32>(prec, static_cast<const float*>(wk.M32), n, sp, nparts, nchunk, wk.Dt, wk.rho_part, s);
    if (parity) launch_parity_sum(wk.rho_part, nchunk, nchunk * n3, n3, n, nparts, rho_all, s);
    else launch_sum_parts(wk.rho_part, nchunk, n3, nparts, rho_all, s);
  } else {
    for (int p = 0; p < nparts; ++p) {
      const int64_t cnt = offs[p + 1] - offs[p];
      double* rho_p = rho_all + p * n3;
      if (cnt == 0) {
        hipLaunchKernelGGL(zero_kernel, dim3(nblk(n3, 256)), dim3(256), 0, s, rho_p, n3);
        continue;
      }
      const float* M32 = wk.M32 ? wk.M32 + 3 * (int64_t)n * offs[p] : nullptr;
      launch_rho_list(prec, M + 3 * (int64_t)n * offs[p], M32, n, (int)cnt, wk, wk.Dt + offs[p], parity, rho_p, s);
    }
  }
  if (parity) {
    hipError_t e = launch_parity_tables(Kx, (int64_t)nparts * nparts * nq, n, s);
    if (e == hipSuccess)
      e = launch_phi_octants(rho_all, nparts, nparts, nparts, Kx, (int64_t)nq * n2, wrep, n, nq, T2_all,
                             (int64_t)nparts * nparts * nq * n3, true, Phi_all, s);
    if (e != hipSuccess) return e;
  } else if (!one) {
    // T1 of box pair (p, q) = rho_q through the tables K^(p,q), at
    // T2_all[(p nparts + q) nq]; Phi_p sums its nparts nq node blocks (the
    // partial grids of rho are free again and hold the node runs' sums)
    const hipError_t e = launch_mode_products(rho_all, (int64_t)nparts * nparts, nparts, Kx, (int64_t)nq * n2, wrep,
                                              n, nq, T2_all, nparts, (int64_t)nparts * nq * n2, nparts * nq, Phi_all,
                                              wk.rho_part, (int64_t)wk.nchunk * n3, s);
    if (e != hipSuccess) return e;
  } else {
    const hipError_t e = launch_phi_grid(rho_all, Kx, wrep, n, nq, wk, Phi_all, s);
    if (e != hipSuccess) return e;
  }
  // The slices of every box's Phi go where the slab products of the mode
  // products were, as many boxes at a time as fit (all of them unless nq = 1
  // meets a coarse grid); a single box has its own room.
  const int64_t ps_box = split_j(prec) ? 2 * n2 * j16_kc(j_slices(prec), n) : 0;
  const int64_t t2_bytes = 8 * n3 * nq * nparts * nparts;
  const int group = one || ps_box == 0 ? nparts : (int)std::max<int64_t>(1, std::min<int64_t>(nparts, t2_bytes / ps_box));
  void* Ps = one || group * ps_box > t2_bytes ? wk.Ps : static_cast<void*>(T2_all);
  for (int p = 0; p < nparts; p += group) {
    const int g = std::min(group, nparts - p);
    int64_t sub[kMaxParts + 1];
    for (int z = 0; z <= g; ++z) sub[z] = offs[p + z] - offs[p];
    if (sub[g] == 0) continue;
    const float* M32 = wk.M32 ? wk.M32 + 3 * (int64_t)n * offs[p] : nullptr;
    launch_projection(prec, M + 3 * (int64_t)n * offs[p], M32, n, sub, g, Phi_all + p * n3, Ps, pairs + offs[p], nb, wk,
                      J, s);
  }
  return hipGetLastError();
}

// Orbitals per launch of the batched orbital densities, and the chunks of
// pairs each orbital's density is split into (the launch holds enough work
// groups for the device either way).
constexpr int kMoBlock = 32;
// The pair contraction runs one work group per compute unit: the chunk
// count is the one between 2 and 4 waves of work groups over the device's
// `cus` units whose last wave is fullest (the first such, at most the
// single-density count).
int mo_chunks(int prec, int n, int npair, int ob, int cus) {
  const int a0g = prec == kFP64 && n <= 48 && !half_tiles(n) ? 16 : 8;
  const int groups = (n + a0g - 1) / a0g * ob;
  const int cap = j_nchunk(prec, n, npair);
  int best = 1;
  double best_eff = -1.0;
  for (int c = (2 * cus + groups - 1) / groups; c <= (4 * cus + groups - 1) / groups && c <= cap; ++c) {
    const int64_t total = (int64_t)groups * c;
    const double eff = (double)total / (double)(((total + cus - 1) / cus) * cus);
    if (eff > best_eff + 1e-9) {
      best_eff = eff;
      best = c;
    }
  }
  if (best_eff < 0) best = cap < (2 * cus + groups - 1) / groups ? cap : (2 * cus + groups - 1) / groups;
  return best < 1 ? 1 : best;
}

size_t mo_work_bytes(int prec, int n, int nq, int npair, int norb, int cus) {
  const size_t n3 = (size_t)n * n * n;
  const int ob = norb < kMoBlock ? norb : kMoBlock;
  return align256(8 * n3 * norb) * 2 + align256(8 * (size_t)npair * ob) +
         align256(8 * n3 * ob * mo_chunks(prec, n, npair, ob, cus)) + align256(8 * n3 * nq * ob);
}

// All orbitals' grid densities rho_i = Q(i,:) M_max (the paper's Q M_max,
// eq. Coul) and Phi_i, in blocks of kMoBlock orbitals with one launch per
// stage for the whole block: the orbital pair densities, the pair
// contraction (grid z = orbital, each orbital's chunks of pairs), the chunk
// sums, the mode products and the node sums; then J_mo(i, j) = <rho_i, Phi_j>.
hipError_t launch_coulomb_mo(int prec, const double* M, int nb, int npair, const int32_t* pairs, int n, int nq,
                             const NodeTables& tb, bool mirrored, const double* Q, int norb, int cus, void* work,
                             double* Jmo, const JWork& w, hipStream_t s) {
  const int64_t n3 = (int64_t)n * n * n;
  const int obmax = norb < kMoBlock ? norb : kMoBlock;
  const bool parity = mirrored && phi_octants(n, obmax);   // obmax tensors a launch
  if (parity) {
    const hipError_t e = launch_parity_tables(tb.K, nq, n, s);
    if (e != hipSuccess) return e;
  }
  convert_moments(prec, M, n, npair, w, s);
  const int nc = mo_chunks(prec, n, npair, obmax, cus);
  char* p = static_cast<char*>(work);
  double* R = reinterpret_cast<double*>(p); p += align256(8 * n3 * norb);
  double* F = reinterpret_cast<double*>(p); p += align256(8 * n3 * norb);
  double* Dt = reinterpret_cast<double*>(p); p += align256(8 * (size_t)npair * obmax);
  double* part = reinterpret_cast<double*>(p); p += align256(8 * n3 * obmax * nc);
  double* T1 = reinterpret_cast<double*>(p);
  for (int i0 = 0; i0 < norb; i0 += obmax) {
    const int ob = norb - i0 < obmax ? norb - i0 : obmax;
    hipLaunchKernelGGL(orbital_pairs_kernel, dim3(nblk(npair, 256), ob), dim3(256), 0, s, Q + (int64_t)i0 * nb, nb,
                       (int64_t)npair, pairs, Dt);
    if (prec == kFP32)
      launch_pair_contraction_rho<JF32>(prec, static_cast<const float*>(w.M32), n, npair, nc, Dt, part, s, ob);
    else launch_pair_contraction_rho<JF64>(prec, M, n, npair, nc, Dt, part, s, ob);
    double* Rb = R + (int64_t)i0 * n3;
    if (parity) {
      // rho and Phi stay in parity form: their dot products are the same
      hipError_t e = launch_parity_sum(part, nc, nc * n3, n3, n, ob, Rb, s);
      if (e == hipSuccess)
        e = launch_phi_octants(Rb, ob, 1, ob, tb.K, 0, tb.w, n, nq, T1, (int64_t)ob * nq * n3, false,
                               F + (int64_t)i0 * n3, s);
      if (e != hipSuccess) return e;
      continue;
    }
    launch_sum_parts(part, nc, n3, ob, Rb, s);
    // the block's mode products on the matrix cores (Phi without 2/sqrt(pi),
    // which the dot products apply)
    // (the partial grids of rho are free again and hold the node runs' sums)
    const hipError_t e = launch_mode_products(Rb, ob, ob, tb.K, 0, tb.w, n, nq, T1, ob, 0, nq,
                                              F + (int64_t)i0 * n3, part, (int64_t)ob * nc * n3, s);
    if (e != hipSuccess) return e;
  }
  // <rho_i, Phi_j> as one product split along the grid (12 orbitals at n = 40:
  // 18 us against 99 us with a work group per pair of orbitals, which read each
  // tensor norb times on norb^2 compute units), where its partials fit in the
  // free partial grids: they do unless a coarse grid meets many orbitals
  const int64_t slice = dot_slice(n3, norb, (int64_t)obmax * nc * n3);
  if (slice > 0) return launch_dot_split(R, F, norb, 1, n3, slice, kTwoOverSqrtPi, part, Jmo, s);
  hipLaunchKernelGGL(mo_dot_kernel, dim3(norb, norb), dim3(256), 0, s, R, F, n3, norb, kTwoOverSqrtPi, Jmo);
  return hipGetLastError();
}


}  // namespace tai
