// Phi = sum_k w_k rho x_0 K_k x_1 K_k x_2 K_k on the n^3 Chebyshev grid, by
// parity.  The grid is symmetric, xi_{n-1-a} = -xi_a, so K(a, b) =
// K(n-1-a, n-1-b) for the plain tables, their truncations to a degree and
// the cross tables of two boxes.  In each mode the sums x_a + x_{n-1-a} and the
// differences x_a - x_{n-1-a} then transform apart, with the ceil(n/2) square
// matrix K_e(i, a) = K(i, a) + K(n-1-i, a) (the row of a middle node once) and
// the floor(n/2) square K_o(i, a) = K(i, a) - K(n-1-i, a).  A grid tensor falls
// into eight octants (sigma_0, sigma_1, sigma_2) of about (n/2)^3 values that
// never mix: half the multiply-adds of every mode product, and an octant and
// its products of one node fit on a compute unit, so that no intermediate
// tensor goes through memory.
//
// A tensor in parity form keeps its n^3 layout: the even component of the
// index pair (a, n-1-a) at a, the odd one at n-1-a (parity_position), so that a
// transform is in place.  The tables in parity form hold, in the place of each
// n x n matrix, K_e and then K_o, transposed: KT[a][i] = K(i, a).
#include "tai_internal.h"

#include <algorithm>

namespace tai {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) double* ConstTable;

inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

constexpr int kOctMaxN = 32;   // largest n of the octant kernel
constexpr int kOctMaxH = 16;

__device__ inline int parity_position(int n, int odd, int a) { return odd ? n - 1 - a : a; }

// Mp[d][.][p] = the parity form of M[d][.][p]; grid (pairs / 256, ceil(n / 2), 3).
__global__ void __launch_bounds__(256)
parity_moments_kernel(const double* __restrict__ M, int n, int64_t npair, double* __restrict__ Mp) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= npair) return;
  const int a = blockIdx.y, b = n - 1 - a;
  const int64_t d0 = (int64_t)blockIdx.z * n * npair + p;
  const double x = M[d0 + a * npair], y = M[d0 + b * npair];
  Mp[d0 + a * npair] = a == b ? x : x + y;
  if (a != b) Mp[d0 + b * npair] = x - y;
}

// One work group per n x n matrix, in place.
__global__ void __launch_bounds__(256) parity_tables_kernel(double* K, int n) {
  __shared__ double s_k[kOctMaxN * kOctMaxN];
  const int nn = n * n, he = (n + 1) / 2, ho = n / 2;
  double* Kk = K + (int64_t)blockIdx.x * nn;
  for (int e = threadIdx.x; e < nn; e += 256) s_k[e] = Kk[e];
  __syncthreads();
  for (int e = threadIdx.x; e < he * he + ho * ho; e += 256) {
    const bool odd = e >= he * he;
    const int h = odd ? ho : he, r = odd ? e - he * he : e;
    const int a = r / h, i = r - a * h;
    const double x = s_k[i * n + a], y = s_k[(n - 1 - i) * n + a];
    Kk[e] = odd ? x - y : (n - 1 - i == i ? x : x + y);
  }
}

// Sums and differences in every mode of eight values at (a_d or n-1-a_d), one
// per lane, bit d of the lane's number choosing the mirrored index of mode d.
// A middle index (its own mirror) has no second value.  The transform is its
// own inverse up to the factor 1/2 per mode and pair of indices that
// phi_octant_kernel applies.
__device__ inline double parity_lanes(double v, int bits, bool mid0, bool mid1, bool mid2) {
  const bool mid[3] = {mid0, mid1, mid2};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double o = __shfl_xor(v, 1 << d);
    const double t = (bits >> d) & 1 ? o - v : v + o;
    v = mid[d] ? v : t;
  }
  return v;
}

// The parity transform of sums of partial tensors: out[y] = transform of
// sum_g part[y ystride + g gstride ..], every sum in a fixed order.  A work group
// owns eight base points (a0, a1, a2) of the lower half of one tensor's grid,
// that is 64 values (lane = 8 point + mirror bits), and splits the parts over
// its waves; npb work groups per tensor.  out may be part when nparts = 1.
template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES)
parity_sum_kernel(const double* part, int nparts, int64_t ystride, int64_t gstride, int n, int npb, int64_t batch,
                  double* out) {
  __shared__ double s_sum[WAVES][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, bits = lane & 7;
  const int he = (n + 1) / 2;
  const int64_t n3 = (int64_t)n * n * n, npoint = (int64_t)he * he * he;
  const int64_t blk = grid_block(), y = blk / npb;
  if (y >= batch) return;
  const int64_t pt = (blk - y * npb) * 8 + (lane >> 3);
  const int a2 = (int)(pt % he), a1 = (int)(pt / he % he), a0 = (int)(pt / ((int64_t)he * he));
  const bool m0 = 2 * a0 == n - 1, m1 = 2 * a1 == n - 1, m2 = 2 * a2 == n - 1;
  const bool in = pt < npoint && !((bits & 1) && m0) && !((bits & 2) && m1) && !((bits & 4) && m2);
  const int64_t at = ((int64_t)parity_position(n, bits & 1, a0) * n + parity_position(n, bits & 2, a1)) * n +
                     parity_position(n, bits & 4, a2);
  const double* src = part + y * ystride + at;
  const int per = (nparts + WAVES - 1) / WAVES;
  const int g0 = wave * per, g1 = min(nparts, g0 + per);
  double v = 0.0;
  if (in) {
#pragma unroll 8
    for (int g = g0; g < g1; ++g) v += src[(int64_t)g * gstride];
  }
  if constexpr (WAVES > 1) {
    s_sum[wave][lane] = v;
    __syncthreads();
    if (wave > 0) return;
    v = 0.0;
#pragma unroll
    for (int q = 0; q < WAVES; ++q) v += s_sum[q][lane];
  }
  v = parity_lanes(v, bits, m0, m1, m2);
  if (in) out[y * n3 + at] = v;
}

// Phi in parity form for n <= 32 (H4 = ceil(ceil(n/2) / 4)).  Grid: rows of 2 T, by
// G along z.  Work group b of eight waves takes the four octants with sigma_0 = b % 2
// of tensor t = b / 2, in LDS, wave w octant w % 4; waves w and w + 4 take the run's
// nodes in turn.  Run z = blockIdx.z takes source
// z / kruns (X[(t nsrc + source) % xmod], tables K + (t nsrc + source) kstride,
// weights w + source nq) and its share of the nodes.  Per node and a0:
//   U = X(a0) K_2^T     H4 MFMAs, X from LDS, the rows a1 and columns i2;
//   V = w_k K_1 U       H4 MFMAs: register s of U holds the rows a1 = 4 s + l/16
//                       at column l % 16, which is the layout of the second
//                       operand, so U never leaves the registers;
//   W(i0) += K_0(i0, a0) V   on the vector units, K_0's column in scalar
//                       registers, W (i0, i1, i2) in the accumulators of the
//                       wave for the whole run.
// The two waves' sums are added through LDS and written, with 1/2 for each
// mode whose index is not the middle one, to run z's block of T tensors.
//   What bounds it: FP64 arithmetic.  The matrix and the vector FP64
// instructions share one pipe (two waves of a SIMD, one of each kind, take the
// sum of their times), so the third product costs the same on either; on the
// vector units its operands V need no transposition.  736 tensors, n = 32,
// 24 nodes: 1060 us, 52 TFLOP/s of the octants' 5.6e10 multiply-adds and adds,
// against 2920 us for the slab and mode-0 kernels, which do twice the arithmetic
// and move 9.2 GB of slab products.  Loading K_0's columns where they are used
// instead of during V's MFMAs: 1157 us.
template <int H4>
__global__ void __launch_bounds__(512, 1)
phi_octant_kernel(const double* __restrict__ X, int64_t T, int nsrc, int64_t xmod, const double* __restrict__ K,
                  int64_t kstride, const double* __restrict__ w, int n, int nq, int kruns, double* __restrict__ Phi) {
  constexpr int HM = 4 * H4, XS = HM + 1, OCT = HM * HM * XS;
  constexpr int kRed = 64 * HM * H4;                     // doubles of one wave's sums
  constexpr int kLds = 4 * OCT > 4 * kRed ? 4 * OCT : 4 * kRed;
  __shared__ __align__(16) double s_x[kLds];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int he = (n + 1) / 2, ho = n / 2;
  const int64_t n2 = (int64_t)n * n, n3 = n2 * n;
  const int64_t t = grid_block() >> 1;
  if (t >= T) return;
  const int sg0 = blockIdx.x & 1, oct = wave & 3, sg1 = oct >> 1, sg2 = oct & 1, half = wave >> 2;
  const int h0 = sg0 ? ho : he, h1 = sg1 ? ho : he, h2 = sg2 ? ho : he;
  const int src = blockIdx.z / kruns, run = blockIdx.z - src * kruns;
  const int64_t ts = t * nsrc + src;
  const int per = (nq + kruns - 1) / kruns, k0 = run * per, k1 = min(nq, k0 + per);

  // the four octants, zero beyond their extents: a column of HM values of a0
  // per thread and step, all its loads in flight
  const double* Xt = X + (ts % xmod) * n3;
  for (int e = threadIdx.x; e < 4 * HM * HM; e += 512) {
    const int o = e / (HM * HM), a1 = e / HM % HM, a2 = e % HM, e1 = o >> 1, e2 = o & 1;
    const bool in = a1 < (e1 ? ho : he) && a2 < (e2 ? ho : he);
    const double* col = Xt + (in ? (int64_t)parity_position(n, e1, a1) * n + parity_position(n, e2, a2) : 0);
    double v[HM];
#pragma unroll
    for (int a0 = 0; a0 < HM; ++a0) v[a0] = in && a0 < h0 ? col[parity_position(n, sg0, a0) * n2] : 0.0;
#pragma unroll
    for (int a0 = 0; a0 < HM; ++a0) s_x[o * OCT + (a0 * HM + a1) * XS + a2] = v[a0];
  }
  __syncthreads();

  double W[HM][H4];
#pragma unroll
  for (int i = 0; i < HM; ++i)
#pragma unroll
    for (int r = 0; r < H4; ++r) W[i][r] = 0.0;

  // fragment s of a table in parity form: K(i = l % 16, a = 4 s + l / 16)
  auto fragment = [&](const double* KT, int h, double scale, double (&f)[H4]) {
#pragma unroll
    for (int s = 0; s < H4; ++s) {
      const int a = 4 * s + kg;
      f[s] = a < h && r16 < h ? scale * KT[a * h + r16] : 0.0;
    }
  };
  const double* Kt = K + ts * kstride;
  const double* ws = w + (int64_t)src * nq;
  const double* xs = s_x + oct * OCT + (r16 < HM ? r16 : HM - 1) * XS + kg;
  double x[H4], c[HM];
  v4d Vp[2];   // V of the previous a0, whose multiply-adds run beside this a0's MFMAs
  // One a0 of node k: U with the previous a0's multiply-adds between the MFMAs,
  // then the operands of the next a0 (x) and of this one's multiply-adds (c, the
  // column a0 of K_0) while the MFMAs of V run.  Entries of c past h0 multiply
  // sums that are not stored; a0 = h0 (h0 odd) is a zero slab.
  auto step = [&](int a0, const double (&f1)[H4], const double (&f2)[H4], ConstTable c0, const v4d& vp, v4d& vn) {
    v4d U = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < H4; ++s) {
      U = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s], f2[s], U, 0, 0, 0);
#pragma unroll
      for (int i = 4 * s; i < 4 * s + 4; ++i)
#pragma unroll
        for (int r = 0; r < H4; ++r) W[i][r] += c[i] * vp[r];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < HM; ++i) c[i] = c0[a0 * h0 + i];
#pragma unroll
    for (int s = 0; s < H4; ++s) x[s] = xs[(a0 + 1 < HM ? a0 + 1 : 0) * (HM * XS) + 4 * s];
    __builtin_amdgcn_sched_barrier(0);
    vn = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < H4; ++s) vn = __builtin_amdgcn_mfma_f64_16x16x4f64(f1[s], U[s], vn, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < HM; ++i) c[i] = 0.0;
  Vp[0] = Vp[1] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int k = k0 + half; k < k1; k += 2) {
    const double* Kk = Kt + (int64_t)k * n2;
    double f1[H4], f2[H4];
    fragment(Kk + (sg1 ? he * he : 0), h1, ws[k], f1);
    fragment(Kk + (sg2 ? he * he : 0), h2, 1.0, f2);
    const ConstTable c0 = (ConstTable)(Kk + (sg0 ? he * he : 0));
#pragma unroll
    for (int s = 0; s < H4; ++s) x[s] = xs[4 * s];
    for (int a0 = 0; a0 < h0; a0 += 2) {
      step(a0, f1, f2, c0, Vp[1], Vp[0]);
      step(a0 + 1, f1, f2, c0, Vp[0], Vp[1]);
    }
  }
#pragma unroll
  for (int i = 0; i < HM; ++i)
#pragma unroll
    for (int r = 0; r < H4; ++r) W[i][r] += c[i] * Vp[1][r];

  // each of the two waves finishes half of the values of i0, the other's half
  // through LDS
  __syncthreads();
  double* red = s_x + oct * kRed + lane;
#pragma unroll
  for (int i = 0; i < HM; ++i)
#pragma unroll
    for (int r = 0; r < H4; ++r)
      if ((i & 1) != half) red[64 * (i * H4 + r)] = W[i][r];
  __syncthreads();
  if (r16 >= h2) return;
  double* out = Phi + ((int64_t)blockIdx.z * T + t) * n3 + parity_position(n, sg2, r16);
  const double c2 = 2 * r16 == n - 1 ? 1.0 : 0.5;
#pragma unroll
  for (int r = 0; r < H4; ++r) {
    const int i1 = kg + 4 * r;
    if (i1 >= h1) continue;
    const double c12 = 2 * i1 == n - 1 ? c2 : 0.5 * c2;
    double* row = out + (int64_t)parity_position(n, sg1, i1) * n;
#pragma unroll
    for (int i = 0; i < HM; ++i)
      if (i < h0 && (i & 1) == half)
        row[parity_position(n, sg0, i) * n2] = (2 * i == n - 1 ? c12 : 0.5 * c12) * (W[i][r] + red[64 * (i * H4 + r)]);
  }
}

}  // namespace

// n = 2 would read the table columns past its last 2 x 2 matrix.  One tensor
// leaves the octants 24 work groups of one node per wave each: J at n = 32
// 85 us against 76 with the slab kernels; two tensors 78 against 83, four 83
// against 97, sixteen 117 against 145 (orbital J), 96 tensors 299 against 473.
// For 9 <= n <= 13 an octant pads its 4 to 7 indices a side to 8, and many tensors,
// which leave no latency to hide, are done sooner by the slab kernels (exchange, 32
// nodes, slabs against octants: n = 9 64 tensors 1.41 of the time, 128 1.18, 400 0.71,
// 800 0.67; n = 13 1.36, 1.03, 0.73, 0.95; n = 14 1.33, 1.05, 0.92, 1.05).
bool phi_octants(int n, int64_t tensors) {
  return n >= 3 && n <= kOctMaxN && tensors >= 2 && (n < 9 || n > 13 || tensors <= 256);
}

hipError_t launch_parity_moments(const double* M, int n, int64_t npair, double* Mp, hipStream_t s) {
  hipLaunchKernelGGL(parity_moments_kernel, dim3(nblk(npair, 256), (n + 1) / 2, 3), dim3(256), 0, s, M, n, npair, Mp);
  return hipGetLastError();
}

hipError_t launch_parity_tables(double* K, int64_t nmat, int n, hipStream_t s) {
  hipLaunchKernelGGL(parity_tables_kernel, dim3((unsigned)nmat), dim3(256), 0, s, K, n);
  return hipGetLastError();
}

hipError_t launch_parity_sum(const double* part, int nparts, int64_t ystride, int64_t gstride, int n, int64_t batch,
                             double* out, hipStream_t s) {
  const int64_t he = (n + 1) / 2;
  const int npb = (int)nblk(he * he * he, 8);
  const dim3 g = grid_rows(npb * batch);
  if (nparts == 1)
    hipLaunchKernelGGL(parity_sum_kernel<1>, g, dim3(64), 0, s, part, nparts, ystride, gstride, n, npb, batch,
                       out);
  else
    hipLaunchKernelGGL(parity_sum_kernel<4>, g, dim3(256), 0, s, part, nparts, ystride, gstride, n, npb, batch, out);
  return hipGetLastError();
}

hipError_t launch_phi_octants(const double* X, int64_t T, int nsrc, int64_t xmod, const double* K, int64_t kstride,
                              const double* w, int n, int nq, double* part, int64_t part_len, bool to_nodes,
                              double* Phi, hipStream_t s) {
  // runs of nodes per source: at least two work groups per compute unit, two
  // nodes per run (one per half of the work group), partial tensors that fit
  const int64_t n3 = (int64_t)n * n * n;
  int64_t kruns = std::min<int64_t>((nq + 1) / 2, (512 + 2 * T * nsrc - 1) / (2 * T * nsrc));
  kruns = std::max<int64_t>(1, std::min(kruns, part_len / (n3 * T * nsrc)));
  const int64_t G = nsrc * kruns;
  double* out = G > 1 ? part : Phi;
  const dim3 g = grid_rows(2 * T, (unsigned)G);
  const int h4 = ((n + 1) / 2 + 3) / 4;
#define TAI_OCT(H)                                                                                                     \
  hipLaunchKernelGGL(phi_octant_kernel<H>, g, dim3(512), 0, s, X, T, nsrc, xmod, K, kstride, w, n, nq, (int)kruns, out)
  if (h4 == 1) TAI_OCT(1);
  else if (h4 == 2) TAI_OCT(2);
  else if (h4 == 3) TAI_OCT(3);
  else TAI_OCT(4);
#undef TAI_OCT
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (to_nodes) return launch_parity_sum(out, (int)G, n3, n3 * T, n, T, Phi, s);
  if (G > 1) launch_sum_parts(out, (int)G, n3 * T, 1, Phi, s);
  return hipGetLastError();
}

}  // namespace tai
