// Assembly of B for few pairs, FP64 and FP32: the contraction of the ring
// kernels (G_{k,d} = M_d^T (K_k M_d), B = (2/sqrt(pi)) sum_k w_k G_{k,0} o
// G_{k,1} o G_{k,2}) with the nodes of one small tile dealt to the waves of a
// work group.
//
// The ring kernels give a work group a panel of 128 to 512 rows and run the
// nodes of each 16-column block in a row.  That shares every Y operand between
// eight waves, but a few hundred pairs make a handful of such blocks, all nodes
// in one chain, and a few thousand make 2 or 3 rounds of them over the device
// with up to a third of the rows below the diagonal.  Here a tile is 16 * RB
// rows by 16 columns, wave w of NW takes nodes w, w + NW, ... with the A operand
// in registers and Y straight from L2 (one direction's fragments refilled as
// soon as they are used, two directions ahead of their next use), and the waves'
// partial tiles meet in LDS.  Two work groups share a compute unit, so one's
// first loads and last sums overlap the other's matrix instructions.
//   What bounds it: the matrix cores (20100 pairs, 24 nodes: FP64 n = 40 66 TFLOP/s,
// FP32 n = 40 110 TFLOP/s), and for a few hundred pairs the loads' latency once
// through.  Moments and B, ring against tiles: 36 pairs, FP64, n = 24, 106 -> 60 us;
// 2080, n = 32, 338 -> 239 us.  Which calls come here is use_tiles' rule
// (tai_api.hip): by pairs and nodes, both kernels measured there.
#include "tai_internal.h"

#include <cmath>
#include <type_traits>

namespace tai {
namespace {

constexpr double kTwoOverSqrtPi = 1.1283791670955126;
constexpr int kTileWaves = 4;
// FP32 sums of at most this many nodes before they go to FP64, as in the ring kernel
constexpr int kGroupT = 8;
constexpr int kXcds = kAsm16Queues;

template <class T>
struct Vec;
template <>
struct Vec<double> {
  typedef double v2 __attribute__((ext_vector_type(2)));
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ inline v4 mma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row of value r of a lane in a 16-row block
  static __device__ inline int row(int kg, int r) { return kg + 4 * r; }
};
template <>
struct Vec<float> {
  typedef float v2 __attribute__((ext_vector_type(2)));
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ inline v4 mma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ inline int row(int kg, int r) { return 4 * kg + r; }
};

// Tiles of the upper triangle in column order: RB columns of 16 share a row
// count, column group g has g + 1 row tiles.
__host__ __device__ inline int tile_total(int npair, int rb) {
  const int ncol = (npair + 15) / 16, g = ncol / rb;
  return rb * (g * (g + 1) / 2) + (ncol % rb) * (g + 1);
}
__device__ inline void tile_at(int t, int rb, int* tr, int* tc) {
  const int u = t / rb;  // g(g+1)/2 <= u < (g+1)(g+2)/2
  int g = (int)((sqrtf(8.0f * (float)u + 1.0f) - 1.0f) * 0.5f);
  while (g * (g + 1) / 2 > u) --g;
  while ((g + 1) * (g + 2) / 2 <= u) ++g;
  const int rem = t - rb * (g * (g + 1) / 2);
  *tc = rb * g + rem / (g + 1);
  *tr = rem % (g + 1);
}

// Call f(integral_constant<int, c>) for the compile-time count c == v (1 <= v <= N).
template <int N, class F>
__device__ inline void with_chunks(int v, F&& f) {
  if constexpr (N == 1) {
    f(std::integral_constant<int, 1>{});
  } else {
    if (v >= N) f(std::integral_constant<int, N>{});
    else with_chunks<N - 1>(v, f);
  }
}

template <class T, int KC, int RB>
__device__ inline void run_tile(const AsmMol& m, int tr, int tc, double (*sums)[16 * RB][17], int* exps) {
  typedef typename Vec<T>::v2 v2;
  typedef typename Vec<T>::v4 v4;
  typedef __attribute__((address_space(1))) const v2 gv2;
  typedef __attribute__((address_space(1))) char gchar;
  constexpr int NCH = KC / 8, NW = kTileWaves;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  // a rectangular block's columns have their own operand rows and exponents
  const bool rect = m.rect != 0;
  const int64_t prow = m.prow, pcol = rect ? (int64_t)m.pcol : prow;
  const int row0 = tr * 16 * RB, col0 = tc * 16;
  const int nq = m.nq;
  const int32_t* __restrict__ nkp = m.nk;
  // one operand fragment per inner chunk of 8: lane l holds inner indices
  // 8 ch + 2 (l / 16) + {0, 1} of row (column) l % 16, of both operands alike
  // (a uniform base and one 32-bit lane offset: no 64-bit address per lane)
  const gchar* A = (const gchar*)m.A + (int64_t)row0 * KC * sizeof(T);
  const gchar* Y = (const gchar*)m.Y + (int64_t)col0 * KC * sizeof(T);
  const uint32_t lo = lane * 2 * (uint32_t)sizeof(T);
  const int64_t dir_a = prow * KC * (int64_t)sizeof(T);  // bytes of one direction's rows
  const int64_t dir_y = pcol * KC * (int64_t)sizeof(T);
  auto load = [&](const gchar* base) { return *(gv2*)(base + lo); };
  constexpr int FB = 128 * sizeof(T);                    // bytes of a fragment
  v2 af[3][RB][NCH], b[3][NCH];
  const int k0 = wave < nq ? wave : nq - 1;
  // summed power-of-two exponents of the tile's rows, then of its columns
  if constexpr (sizeof(T) == 4) {
    if (threadIdx.x < 16 * RB + 16) {
      const bool row = threadIdx.x < 16 * RB;
      const int32_t* __restrict__ ex = row || !rect ? m.ex : m.exc;
      const int64_t p = row ? prow : pcol, i = row ? row0 + threadIdx.x : col0 + (threadIdx.x - 16 * RB);
      exps[threadIdx.x] = ex[i] + ex[p + i] + ex[2 * p + i] - (row ? m.ysh : 0);
    }
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) b[d][ch] = load(Y + (k0 * 3 + d) * dir_y + FB * ch);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) af[d][rb][ch] = load(A + d * dir_a + FB * (rb * NCH + ch));
  }
  v4 acc[RB];
  double sum[RB][4];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    acc[rb] = v4{0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[rb][r] = 0.0;
  }
  int left = kGroupT;
  // inner chunks of a node's degree
  auto chunks_of = [&](int k) { return nkp ? (nkp[k] + 7) / 8 : NCH; };
  int nch = chunks_of(k0);
  for (int k = wave; k < nq; k += NW) {
    const int kn = k + NW < nq ? k + NW : k;  // node of the next loads
    const int nch_next = chunks_of(kn);
    // straight code for each chunk count, so that the loads of the next node
    // stay in flight over this one's matrix instructions
    with_chunks<NCH>(nch, [&](auto nc) {
      constexpr int NC = decltype(nc)::value;
      v4 H[RB], G[RB];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int ch = 0; ch < NC; ++ch)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              G[rb] = Vec<T>::mma(af[d][rb][ch][j], b[d][ch][j], ch + j == 0 ? v4{0, 0, 0, 0} : G[rb]);
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) b[d][ch] = load(Y + (kn * 3 + d) * dir_y + FB * ch);
        __builtin_amdgcn_sched_barrier(0);  // or the loads wait for the end of the node
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          if (d == 0) H[rb] = G[rb];
          else if (d == 1) H[rb] *= G[rb];
          else acc[rb] += H[rb] * G[rb];
        }
      }
      __asm__ volatile("; %0 chunks" ::"n"(NC));  // no common tail of the forms
    });
    nch = nch_next;
    if constexpr (sizeof(T) == 4) {
      if (--left == 0 || k + NW >= nq) {
        left = kGroupT;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
          for (int r = 0; r < 4; ++r) sum[rb][r] += (double)acc[rb][r];
          acc[rb] = v4{0, 0, 0, 0};
        }
      }
    }
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      sums[wave][16 * rb + Vec<T>::row(kg, r)][r16] = sizeof(T) == 4 ? sum[rb][r] : (double)acc[rb][r];
  __syncthreads();
  const int nrow = m.npair, ncol = rect ? m.ncol : m.npair;
  const int64_t ldb = m.ldb;
  T* __restrict__ B = static_cast<T*>(m.B);
  T* __restrict__ Bt = static_cast<T*>(rect ? m.Bt : m.B);
  // entries kept: rows row <= col and their mirror row < col; of a rectangular
  // block every one of both
  const int over = rect ? nrow : 0;
  auto entry = [&](int i, int j) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += sums[w][i][j];
    v *= kTwoOverSqrtPi;
    if constexpr (sizeof(T) == 4) v = ldexp(v, exps[i] + exps[16 * RB + j]);
    return (T)v;
  };
  // rows of 16 entries (row <= col), then the mirrored rows (row < col)
#pragma unroll
  for (int u = 0; u < RB; ++u) {
    const int i = 16 * u + (threadIdx.x >> 4), j = threadIdx.x & 15;
    if (col0 + j < ncol && row0 + i < nrow && row0 + i <= col0 + j + over)
      B[(int64_t)(row0 + i) * ldb + col0 + j] = entry(i, j);
  }
#pragma unroll
  for (int u = 0; u < RB; ++u) {
    const int e = threadIdx.x + 64 * NW * u;
    const int i = e % (16 * RB), j = e / (16 * RB);
    if (col0 + j < ncol && row0 + i < nrow && row0 + i < col0 + j + over)
      Bt[(int64_t)(col0 + j) * ldb + row0 + i] = entry(i, j);
  }
}

// Each XCD takes one contiguous eighth of the tiles in column order, so that the
// work groups sharing an L2 share their columns' Y.
__device__ inline int xcd_tile(int b, int total) {
  const int per = (total + kXcds - 1) / kXcds;
  const int t = (b % kXcds) * per + b / kXcds;
  return b < kXcds * per && t < total ? t : -1;
}

// One molecule (m), or a batch (mols): molecule i owns the tiles from its tile0 up
// to the next one's (none of a molecule that the ring kernel takes).  Rows of the
// grid (grid_rows): the tiles of a batch with 70 GB of B pass 2^32 threads.
template <class T, int KC, int RB>
__global__ void __launch_bounds__(64 * kTileWaves, 2)
assemble_tiles_kernel(AsmMol m, const AsmMol* __restrict__ mols, int nmol, int total) {
  __shared__ double sums[kTileWaves][16 * RB][17];
  __shared__ int exps[16 * RB + 16];
  int t = xcd_tile((int)grid_block(), total);
  if (t < 0) return;
  if (mols) {
    int lo = 0, hi = nmol - 1;  // the last molecule with tile0 <= t
    while (lo < hi) {
      const int mid = (lo + hi + 1) / 2;
      if (mols[mid].tile0 <= t) lo = mid;
      else hi = mid - 1;
    }
    m = mols[lo];
    t -= (int)m.tile0;
  }
  int tr, tc;
  if (m.rect) {
    const int nr = (m.npair + 16 * RB - 1) / (16 * RB);
    tc = t / nr;
    tr = t - tc * nr;
  } else {
    tile_at(t, RB, &tr, &tc);
  }
  run_tile<T, KC, RB>(m, tr, tc, sums, exps);
}

// Row blocks of the larger tile: while the A operand (12 VGPRs of FP64 per row
// block and chunk, 6 of FP32) leaves room for the fragments on their way.
template <class T>
constexpr int max_rb(int kc) { return sizeof(T) == 4 ? (kc <= 40 ? 4 : 2) : (kc <= 40 ? 2 : 1); }

template <class T, int KC, int RB>
hipError_t launch_one(const AsmMol& m, const AsmMol* mols_dev, int nmol, int total, hipStream_t s) {
  static_assert(kGridRow % kXcds == 0, "a work group's number gives its XCD in every row");
  const dim3 grid = grid_rows((int64_t)kXcds * ((total + kXcds - 1) / kXcds)), block(64 * kTileWaves);
  hipLaunchKernelGGL((assemble_tiles_kernel<T, KC, RB>), grid, block, 0, s, m, mols_dev, nmol, total);
  return hipGetLastError();
}

template <class T, int KC>
hipError_t launch_kc(int rb, const AsmMol& m, const AsmMol* mols_dev, int nmol, int total, hipStream_t s) {
  if (rb == 1) return launch_one<T, KC, 1>(m, mols_dev, nmol, total, s);
  if constexpr (max_rb<T>(KC) > 1)
    if (rb == max_rb<T>(KC)) return launch_one<T, KC, max_rb<T>(KC)>(m, mols_dev, nmol, total, s);
  return hipErrorInvalidValue;
}

template <class T>
hipError_t launch_type(int kc, int rb, const AsmMol& m, const AsmMol* mols_dev, int nmol, int total, hipStream_t s) {
  switch (kc) {
    case 8: return launch_kc<T, 8>(rb, m, mols_dev, nmol, total, s);
    case 16: return launch_kc<T, 16>(rb, m, mols_dev, nmol, total, s);
    case 24: return launch_kc<T, 24>(rb, m, mols_dev, nmol, total, s);
    case 32: return launch_kc<T, 32>(rb, m, mols_dev, nmol, total, s);
    case 40: return launch_kc<T, 40>(rb, m, mols_dev, nmol, total, s);
    case 48: return launch_kc<T, 48>(rb, m, mols_dev, nmol, total, s);
  }
  if constexpr (sizeof(T) == 4) {
    if (kc == 56) return launch_kc<T, 56>(rb, m, mols_dev, nmol, total, s);
    if (kc == 64) return launch_kc<T, 64>(rb, m, mols_dev, nmol, total, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int asm_tile_count(const AsmMol& m, int rb) {
  return m.rect ? (m.npair + 16 * rb - 1) / (16 * rb) * ((m.ncol + 15) / 16) : tile_total(m.npair, rb);
}
int asm_tiles_max_rb(int prec, int kc) { return prec == kFP64 ? max_rb<double>(kc) : max_rb<float>(kc); }

hipError_t launch_assemble_tiles(int prec, int kc, int rb, const AsmMol& m, hipStream_t s) {
  const int total = asm_tile_count(m, rb);
  return prec == kFP64 ? launch_type<double>(kc, rb, m, nullptr, 1, total, s)
                       : launch_type<float>(kc, rb, m, nullptr, 1, total, s);
}

hipError_t launch_assemble_tiles_batch(int prec, int kc, int rb, const AsmMol* mols_dev, int nmol, int total,
                                       hipStream_t s) {
  return prec == kFP64 ? launch_type<double>(kc, rb, AsmMol{}, mols_dev, nmol, total, s)
                       : launch_type<float>(kc, rb, AsmMol{}, mols_dev, nmol, total, s);
}

}  // namespace tai
