// 1D moments of basis pairs against the Lagrange basis on the Chebyshev
// nodes (eq. defV in node form), FP64:
//
//   M[d][a][p] = int_{-L}^{L} g_{mu,d}(x) g_{nu,d}(x) l_a(x) dx.
//
// By the Gaussian product rule (Prop. 2.1, eq. gauss_prod) the integrand is
//   N N' (x-A)^l (x-B)^l' E exp(-p (x-P)^2),  p = a+b, P = (aA+bB)/p,
//   E = exp(-ab/p (A-B)^2).
// One thread owns one (pair, direction) and accumulates the Chebyshev moments
// int f(x) T_k(x/L) dx by the three-term recurrence -- the paper's own W
// matrices of eq. defV in the T_k basis -- over the points of a quadrature
// rule, then maps them to the Lagrange basis with the fixed n x n matrix gam.
// Two rules (see kHermiteCut):
//   * the Gaussian lies inside the box: Gauss-Hermite of order (NMAX + 8) / 2,
//     exact for the polynomial (x-A)^l (x-B)^l' T_k of degree <= NMAX + 7,
//     with no exponential per point;
//   * it reaches the box's edge: composite Gauss-Legendre, 4 panels of 24 (28
//     beyond 48 nodes) points, over the part of the box where the Gaussian is above e^-56 of
//     its largest value in the box (kLegendreCut).
#include "tai_internal.h"
#include "tai_device.h"

#include <algorithm>

#include <cmath>
#include <type_traits>

namespace tai {
namespace {

__device__ inline double norm_1d(double a, int l) {
  // [(2a/pi)^(1/2) (4a)^l / (2l-1)!!]^(1/2)
  double df = 1.0;
  for (int k = 2 * l - 1; k > 0; k -= 2) df *= k;
  double p4 = 1.0;
  for (int k = 0; k < l; ++k) p4 *= 4.0 * a;
  return sqrt(sqrt(2.0 * a / M_PI) * p4 / df);
}

// Gauss-Hermite rules on the whole axis, int exp(-y^2) f(y) dy = sum w f(y):
// the positive nodes (the rule is symmetric, every order even), from Newton's
// method on the orthonormal Hermite recurrence in 60 digits, the weights
// 1 / sum_j h_j(y)^2.
__constant__ double kHermY[] = {
    // order 12
    0.31424037625435913, 0.9477883912401638, 1.5976826351526048, 2.2795070805010598, 3.0206370251208896,
    3.889724897869782,
    // order 16
    0.27348104613815244, 0.8229514491446559, 1.3802585391988809, 1.9517879909162539, 2.5462021578474814,
    3.176999161979956, 3.869447904860123, 4.688738939305819,
    // order 20
    0.24534070830090124, 0.7374737285453944, 1.234076215395323, 1.7385377121165861, 2.2549740020892757,
    2.7888060584281305, 3.3478545673832163, 3.944764040115625, 4.603682449550744, 5.387480890011233,
    // order 24
    0.22441454747251557, 0.6741711070372123, 1.1267608176112451, 1.5842500109616942, 2.049003573661699,
    2.5238810170114268, 3.0125461375655647, 3.5200068130345246, 4.05366440244815, 4.625662756423787,
    5.259382927668044, 6.01592556142574,
    // order 28
    0.20806738269073688, 0.6248367195052092, 1.0435352737542083, 1.465537263457409, 1.8923604968376853,
    2.325749842656441, 2.767795352913594, 3.2211120765614556, 3.6891342384616794, 4.1766367421292685,
    4.690756523943118, 5.243285373202936, 5.85701464138285, 6.591605442367743,
    // order 36
    0.1838533671058128, 0.5519014332904228, 0.9209818015707532, 1.291810958820924, 1.6651500018434144,
    2.04182718355442, 2.4227660420535617, 2.8090222351311036, 3.2018339457881586, 3.6026938571484757,
    4.01345656774947, 4.436506970192857, 4.875039972467084, 5.333560107113064, 5.818863279505577,
    6.342243330994412, 6.925598990259942, 7.6263257540038945,
};
__constant__ double kHermW[] = {
    // order 12
    0.5701352362624795, 0.26049231026416114, 0.05160798561588393, 0.0039053905846290616,
    8.573687043587859e-05, 2.658551684356302e-07,
    // order 16
    0.5079294790166138, 0.2806474585285337, 0.08381004139898583, 0.012880311535509973,
    0.0009322840086241805, 2.7118600925378814e-05, 2.3209808448652107e-07, 2.6548074740111823e-10,
    // order 20
    0.4622436696006101, 0.28667550536283415, 0.10901720602002332, 0.024810520887463612,
    0.003243773342237862, 0.00022833863601635397, 7.802556478532063e-06, 1.0860693707692817e-07,
    4.3993409922731804e-10, 2.2293936455341513e-13,
    // order 24
    0.4269311638686992, 0.286179535346443, 0.12773962178455917, 0.03744547050323074, 0.007048355810072671,
    0.0008236924826884174, 5.68869163640438e-05, 2.1582457049023337e-06, 4.0189711749414294e-08,
    3.046254269987564e-10, 6.58462024307817e-13, 1.664368496489109e-16,
    // order 28
    0.39860471782645146, 0.28256139125938873, 0.14139460978695492, 0.04951488928989814, 0.01196842321435482,
    0.0019573312944089895, 0.00021061810002403233, 1.4345504229714415e-05, 5.857719720992981e-07,
    1.3256825015417078e-08, 1.4758531682776886e-10, 6.639436714909664e-13, 8.31593795120683e-16,
    1.1401393479036762e-19,
    // order 36
    0.35554007427370876, 0.27170124700952747, 0.15835545375116658, 0.07010475010517768,
    0.023425767509731767, 0.005856425986559559, 0.0010825347566868026, 0.00014569615962636061,
    1.3997029220328964e-05, 9.355570089773252e-07, 4.207491323109071e-08, 1.2178678209557233e-09,
    2.1353541817845545e-11, 2.0809126742868742e-13, 9.902901686906338e-16, 1.8615979878080026e-18,
    9.25640308355832e-22, 4.44715341757558e-26,
};
// Gauss-Legendre rules on [-1, 1], the positive nodes and their weights, from
// Newton's method on the Legendre recurrence in 50 digits.
__constant__ double kLegY[] = {
    // order 24
    0.06405689286260563, 0.1911188674736163, 0.3150426796961634, 0.4337935076260451, 0.5454214713888396,
    0.6480936519369755, 0.7401241915785544, 0.820001985973903, 0.8864155270044011, 0.9382745520027328,
    0.9747285559713095, 0.9951872199970213,
    // order 28
    0.05507928988403427, 0.16456928213338076, 0.2720616276351781, 0.3762515160890787, 0.4758742249551183,
    0.5697204718114017, 0.656651094038865, 0.7356108780136318, 0.8056413709171791, 0.8658925225743951,
    0.9156330263921321, 0.9542592806289382, 0.9813031653708727, 0.9964424975739544,
};
__constant__ double kLegW[] = {
    // order 24
    0.12793819534675216, 0.1258374563468283, 0.12167047292780339, 0.1155056680537256, 0.10744427011596563,
    0.09761865210411388, 0.08619016153195327, 0.0733464814110803, 0.05929858491543678, 0.04427743881741981,
    0.028531388628933663, 0.0123412297999872,
    // order 28
    0.1100470130164752, 0.10871119225829413, 0.10605576592284642, 0.10211296757806076, 0.09693065799792992,
    0.09057174439303284, 0.08311341722890121, 0.07464621423456878, 0.0652729239669996, 0.05510734567571675,
    0.04427293475900423, 0.03290142778230438, 0.02113211259277126, 0.009124282593094517,
};

// first entry of Gauss-Hermite order `m` in the tables above
constexpr int hermite_offset(int m) {
  int o = 0;
  for (int k : {12, 16, 20, 24, 28, 36}) {
    if (k == m) return o;
    o += k / 2;
  }
  return -1;
}

// A pair takes the Gauss-Hermite rule in a direction when its Gaussian factor
// keeps this many 1/sqrt(p) of room on both sides inside [-L, L].  The rule
// integrates the polynomial over the whole axis; what lies beyond the box falls
// off as exp(-64) and less while T_k grows as cosh(k acosh(x / L)).  Against the
// integral of the factor's absolute value, with exactly this room and the worst
// l + l' <= 8, the part beyond is 9e-20 at k = 39, 2e-18 at k = 48 and 1e-15 at
// k = 63.  (Nodes reach 7.63 for the largest order, so T_k stays bounded at all
// of them.)  Against 64-bit-mantissa references the rule's
// error over the range of exponents is at most that of the composite rule.
constexpr double kHermiteCut = 8.0;

// The composite Gauss-Legendre rule's interval ends where the Gaussian falls
// below exp(-kLegendreCut^2) of its largest value inside the box (and
// 9/sqrt(p) from the centre at most, where a centre outside the box leaves
// nothing).  Largest error of a column over its integral of |f|, against
// 64-bit mantissas and 24 x 64 points, random pairs with l + l' <= 8: 4 x 24
// points to P +- 9/sqrt(p) 2.5e-12, 2.1e-11, 5.4e-9 at n = 40, 48, 64; 4 x 24
// to this cut 8e-14 and 1.8e-13 at n = 40 and 48, 4 x 28 1.0e-13 at n = 64
// (rounding alone: 7e-14).
constexpr double kLegendreCut = 7.5;

constexpr int kMomThreads = 256;
// waves per SIMD that the moments in registers leave room for
constexpr int moment_waves(int nmax) { return nmax <= 16 ? 4 : nmax <= 48 ? 3 : 2; }

// x of the lane whose number differs in bit 0 (kCtrl 0xB1) or bit 1 (0x4E)
template <int kCtrl>
__device__ inline double quad_swap(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), kCtrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), kCtrl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// What bounds it: FP64 VALU.  A work group takes kMomThreads items (pair,
// direction), sorts them by rule, and runs each rule on full waves: the pairs
// of one diffuse function with all others mix the rules lane by lane, and a
// wave that ran both would pay for both.
//   Gauss-Hermite: a thread per item, NMAX + 8 points' worth of recurrence
// halved by taking +y and -y together; about NMAX (NMAX + 8) multiply-adds
// and NMAX^2 / 2 for the map to the nodes, whose matrix comes through the
// scalar cache (from LDS, a broadcast read per one or two multiply-adds took
// longer than the arithmetic).
//   Gauss-Legendre: four lanes per item, a panel each, added across the four
// in a fixed order; four times the points cost no more time in a group
// with few such items (a thread per item left a small molecule's single wave
// with 96 points and exponentials in a row).
// The map uses gam[n-1-a][k] = (-1)^k gam[a][k]: two rows from one pass.
//   Measured, against the composite rule with a thread per item: 186355 pairs
// at n = 48 369 -> 144 us (0.21 GB written), 80200 pairs at n = 40 169 -> 71 us,
// 64 molecules of 20 .. 120 functions at n = 32 311 -> 151 us; one molecule's
// 36 pairs 33 -> 22 us, where one wave's chain of instructions is the time.
template <int NMAX>
__device__ inline void moments_body(const DevBasis& bs, int n, double L, const NodeTables& tb,
                                    double* __restrict__ M, int64_t npair, const int32_t* __restrict__ pairs = nullptr) {
  constexpr int kWaves = kMomThreads / 64;
  constexpr int kGS = NMAX + 2;            // LDS row stride: a quad's four rows start in different banks
  __shared__ int s_item[kMomThreads];
  __shared__ int s_cnt[kWaves];
  __shared__ __align__(16) double s_gam[NMAX / 2 * kGS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * kMomThreads;
  if (base >= 3 * npair) return;
  const double invL = 1.0 / L;

  // one item: column p of direction d, its Gaussian product
  struct Item {
    int64_t p;
    int d, la, lb;
    double pp, P, A, B, pref;
  };
  // column p is pair pairs[p] of the full list when a screened list is given
  // (entries outside it give zero moments)
  auto item = [&](int64_t g) {
    Item it;
    it.d = (int)(g / npair);
    it.p = g - it.d * npair;
    int64_t gp = it.p;
    bool valid = true;
    if (pairs) {
      gp = pairs[it.p];
      valid = gp >= 0 && gp < (int64_t)bs.nb * (bs.nb + 1) / 2;
      if (!valid) gp = 0;
    }
    int mu, nu;
    decode_pair(bs.nb, gp, mu, nu);
    const int d = it.d;
    const double a = bs.alpha[mu], b = bs.alpha[nu];
    it.A = bs.center[3 * mu + d];
    it.B = bs.center[3 * nu + d];
    it.la = bs.lxyz[3 * mu + d];
    it.lb = bs.lxyz[3 * nu + d];
    double nrm;
    if (bs.coef) {
      nrm = (d == 0) ? bs.coef[mu] * bs.coef[nu] : 1.0;
    } else {
      nrm = norm_1d(a, it.la) * norm_1d(b, it.lb);
    }
    it.pp = a + b;
    it.P = (a * it.A + b * it.B) / it.pp;
    const double E = exp(-a * b / it.pp * (it.A - it.B) * (it.A - it.B));
    it.pref = valid ? nrm * E : 0.0;
    return it;
  };
  auto inside = [&](double pp, double P) {
    const double room = kHermiteCut / sqrt(pp);
    return P - room >= -L && P + room <= L;
  };
  // (x - A)^la (x - B)^lb, the powers 0 .. 4 by selects
  auto powers = [](const Item& it, double x) {
    const double xa = x - it.A, xb = x - it.B;
    double r = 1.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (__any(it.la > k)) r *= it.la > k ? xa : 1.0;
      if (__any(it.lb > k)) r *= it.lb > k ? xb : 1.0;
    }
    return r;
  };
  // adds f0 T_k(u0) + f1 T_k(u1) to mom[k]
  auto add_two = [](double (&mom)[NMAX], double u0, double f0, double u1, double f1) {
    const double v0 = 2.0 * u0, v1 = 2.0 * u1;
    double s0 = 1.0, t0 = u0, s1 = 1.0, t1 = u1;
    mom[0] += f0 + f1;
    mom[1] += f0 * u0 + f1 * u1;
#pragma unroll
    for (int k = 2; k < NMAX; ++k) {
      const double r0 = v0 * t0 - s0, r1 = v1 * t1 - s1;
      mom[k] += f0 * r0;
      mom[k] += f1 * r1;
      s0 = t0; t0 = r0;
      s1 = t1; t1 = r1;
    }
  };

  // items in range, Gauss-Hermite ones first (stable)
  const int count = (int)(3 * npair - base < kMomThreads ? 3 * npair - base : kMomThreads);
  bool herm = false;
  if (tid < count) {
    const Item it = item(base + tid);
    herm = inside(it.pp, it.P);
  }
  const uint64_t hm = __ballot(herm);
  if (lane == 0) s_cnt[wave] = __popcll(hm);
  __syncthreads();
  int before = 0, nherm = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    before += w < wave ? s_cnt[w] : 0;
    nherm += s_cnt[w];
  }
  const int rank = before + __popcll(hm & __lanemask_lt());
  s_item[herm ? rank : nherm + tid - rank] = tid;
  if (nherm < count) {                     // the other rule's rows of gam
    for (int e = tid; e < (n + 1) / 2 * kGS; e += kMomThreads) {
      const int a = e / kGS, k = e - a * kGS;
      s_gam[e] = k < n ? tb.gam[a * n + k] : 0.0;
    }
  }
  __syncthreads();

  double mom[NMAX];
  if (tid < nherm) {
    const Item it = item(base + s_item[tid]);
    constexpr int kOrder = (NMAX + 8) / 2, kOff = hermite_offset(kOrder);
    static_assert(kOff >= 0, "no Gauss-Hermite rule of this order");
    const double rs = 1.0 / sqrt(it.pp), ps = it.pref * rs;
#pragma unroll
    for (int k = 0; k < NMAX; ++k) mom[k] = 0.0;
#pragma unroll 1
    for (int i = 0; i < kOrder / 2; ++i) {
      const double dx = kHermY[kOff + i] * rs, wt = kHermW[kOff + i] * ps;
      const double x0 = it.P + dx, x1 = it.P - dx;
      add_two(mom, x0 * invL, wt * powers(it, x0), x1 * invL, wt * powers(it, x1));
    }
    // rows of gam are read NMAX long: the moments beyond n count as zero
    // there (the table is followed by finite values, see launch_nodes)
#pragma unroll
    for (int k = 0; k < NMAX; ++k)
      if (k >= n) mom[k] = 0.0;
    typedef const __attribute__((address_space(4))) double* ConstTable;
    double* out = M + (int64_t)it.d * n * npair + it.p;
#pragma unroll 1
    for (int a = 0; 2 * a < n; ++a) {
      const ConstTable gr = (ConstTable)(tb.gam + a * n);
      double even = 0.0, odd = 0.0;
#pragma unroll
      for (int k = 0; k < NMAX; k += 2) {
        even += gr[k] * mom[k];
        odd += gr[k + 1] * mom[k + 1];
      }
      out[(int64_t)a * npair] = even + odd;
      if (n - 1 - a > a) out[(int64_t)(n - 1 - a) * npair] = even - odd;
    }
  }

#pragma unroll 1
  for (int c0 = nherm; c0 < count; c0 += kMomThreads / 4) {
    if (c0 + (wave << 4) >= count) break;  // whole waves
    const int slot = c0 + (tid >> 2), panel = tid & 3;
    const Item it = item(base + s_item[slot < count ? slot : count - 1]);
    constexpr int kHalf = NMAX > 48 ? 14 : 12, kOff = NMAX > 48 ? 12 : 0;
    const double rp = sqrt(it.pp), past = fmax(0.0, fabs(it.P) - L) * rp;
    const double half = fmin(9.0, sqrt(kLegendreCut * kLegendreCut + past * past)) / rp;
    const double lo = fmax(-L, it.P - half);
    const double hi = fmin(L, it.P + half);
    const double h = (hi > lo) ? 0.125 * (hi - lo) : 0.0;   // half a panel
    const double mid = lo + (2 * panel + 1) * h;
#pragma unroll
    for (int k = 0; k < NMAX; ++k) mom[k] = 0.0;
#pragma unroll 1
    for (int j = 0; j < kHalf; ++j) {
      const double dx = h * kLegY[kOff + j], wt = it.pref * (h * kLegW[kOff + j]);
      const double x0 = mid + dx, x1 = mid - dx, d0 = x0 - it.P, d1 = x1 - it.P;
      add_two(mom, x0 * invL, wt * powers(it, x0) * exp(-it.pp * d0 * d0), x1 * invL,
              wt * powers(it, x1) * exp(-it.pp * d1 * d1));
    }
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
      mom[k] += quad_swap<0xB1>(mom[k]);
      __asm__ volatile("" : "+v"(mom[k]));   // one after another: all at once would double the registers
    }
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
      mom[k] += quad_swap<0x4E>(mom[k]);
      __asm__ volatile("" : "+v"(mom[k]));   // one after another: all at once would double the registers
    }
    if (slot >= count) continue;
    double* out = M + (int64_t)it.d * n * npair + it.p;
#pragma unroll 1
    for (int a = panel; 2 * a < n; a += 4) {
      const double* gr = s_gam + a * kGS;
      double even = 0.0, odd = 0.0;
#pragma unroll
      for (int k = 0; k < NMAX; k += 2) {
        even += gr[k] * mom[k];
        odd += gr[k + 1] * mom[k + 1];
      }
      out[(int64_t)a * npair] = even + odd;
      if (n - 1 - a > a) out[(int64_t)(n - 1 - a) * npair] = even - odd;
    }
  }
}

template <int NMAX>
__global__ void __launch_bounds__(kMomThreads, moment_waves(NMAX))
moments_kernel(DevBasis bs, int n, double L, NodeTables tb, double* __restrict__ M, int64_t npair,
               const int32_t* __restrict__ pairs) {
  moments_body<NMAX>(bs, n, L, tb, M, npair, pairs);
}

// Screening (section 6.3, compression by screening).  One wave per row mu of
// the pair list counts, then writes, the pairs (mu, nu >= mu) whose Gaussian
// product prefactor exp(-ab/(a+b) |A - B|^2) exceeds tau, 64 columns nu at a
// time: a ballot of the lanes that keep their pair gives each kept lane its
// slot (the kept lanes below it) and the chunk's count.  A single work group
// turns the row counts into offsets in between, so the kept indices come out
// in ascending order.  The exponent is formed with unfused, left-to-right
// operations.
__device__ inline bool keep_pair(const DevBasis& bs, double tau, int mu, int nu) {
#pragma clang fp contract(off)
  const double a = bs.alpha[mu], b = bs.alpha[nu];
  double r2 = 0.0;
  for (int d = 0; d < 3; ++d) {
    const double x = bs.center[3 * mu + d] - bs.center[3 * nu + d];
    r2 = r2 + x * x;
  }
  const double e = (a * b) / (a + b) * r2;
  return tau <= 0.0 || exp(-e) > tau;
}

constexpr int kScreenRows = 4;  // rows (one wave each) per work group
constexpr int kScreenThreads = 64 * kScreenRows;

__global__ void __launch_bounds__(kScreenThreads) screen_count_kernel(DevBasis bs, double tau, int32_t* rows) {
  const int mu = blockIdx.x * kScreenRows + threadIdx.x / 64;
  const int lane = threadIdx.x % 64;
  if (mu >= bs.nb) return;  // whole waves
  int c = 0;
  for (int nu0 = mu; nu0 < bs.nb; nu0 += 64) {
    const int nu = nu0 + lane;
    c += __popcll(__ballot(nu < bs.nb && keep_pair(bs, tau, mu, nu)));
  }
  if (lane == 0) rows[mu] = c;
}

// exclusive scan of rows[0 .. nb) in place, total to rows[nb] and *count
__global__ void __launch_bounds__(1024) screen_scan_kernel(int nb, int32_t* rows, int32_t* count) {
  __shared__ int32_t part[1024];
  const int t = threadIdx.x, per = (nb + 1023) / 1024;
  const int lo = min(nb, t * per), hi = min(nb, lo + per);
  int32_t sum = 0;
  for (int i = lo; i < hi; ++i) sum += rows[i];
  part[t] = sum;
  __syncthreads();
  if (t == 0) {
    int32_t acc = 0;
    for (int i = 0; i < 1024; ++i) {
      const int32_t v = part[i];
      part[i] = acc;
      acc += v;
    }
    rows[nb] = acc;
    *count = acc;
  }
  __syncthreads();
  int32_t acc = part[t];
  for (int i = lo; i < hi; ++i) {
    const int32_t v = rows[i];
    rows[i] = acc;
    acc += v;
  }
}

__global__ void __launch_bounds__(kScreenThreads)
screen_write_kernel(DevBasis bs, double tau, const int32_t* __restrict__ rows, int32_t* __restrict__ pairs) {
  const int mu = blockIdx.x * kScreenRows + threadIdx.x / 64;
  const int lane = threadIdx.x % 64;
  if (mu >= bs.nb) return;  // whole waves
  int32_t o = rows[mu];
  const uint64_t below = __lanemask_lt();
  const int64_t p0 = pair_row_start(bs.nb, mu);
  for (int nu0 = mu; nu0 < bs.nb; nu0 += 64) {
    const int nu = nu0 + lane;
    const bool k = nu < bs.nb && keep_pair(bs, tau, mu, nu);
    const uint64_t m = __ballot(k);
    if (k) pairs[o + __popcll(m & below)] = (int32_t)(p0 + (nu - mu));
    o += __popcll(m);
  }
}

// blockIdx.y = partition z of the adaptive boxes: pairs pairs[off[z] ..),
// box half-width L[z], moment block M + 3 n off[z].  Only L depends on the
// box (the node map does not), so one launch serves all boxes;
// blocks past a partition's 3 count threads return as a whole.
template <int NMAX>
__global__ void __launch_bounds__(kMomThreads, moment_waves(NMAX))
moments_parts_kernel(DevBasis bs, int n, PartSpans sp, NodeTables tb, double* __restrict__ M,
                     const int32_t* __restrict__ pairs) {
  const int z = blockIdx.y;
  const int64_t o = sp.off[z], cnt = sp.off[z + 1] - o;
  if ((int64_t)blockIdx.x * kMomThreads >= 3 * cnt) return;
  moments_body<NMAX>(bs, n, sp.L[z], tb, M + 3 * (int64_t)n * o, cnt, pairs + o);
}

// blockIdx.y = molecule; blocks past a molecule's 3*npair items return
template <int NMAX>
__global__ void __launch_bounds__(kMomThreads, moment_waves(NMAX))
moments_batch_kernel(const PrepMol* __restrict__ mols, int n) {
  const PrepMol& m = mols[blockIdx.y];
  // copies: the descriptor could alias the moments written
  const DevBasis bs = m.basis;
  const NodeTables tb = m.tb;
  moments_body<NMAX>(bs, n, m.L, tb, m.M, m.npair);
}

// Coefficient moments mu_d[j][p] = sum_a T_j(xi_a / L) M_d[a][p], the
// moments against T_j (j < n) that the per-node degree form contracts (eq.
// tensors with the nested moments of section 3.2): T_j = sum_a T_j(xi_a) l_a
// for every j < n.  One thread per (pair, direction).  T_j is even or odd, so
// mu_j takes the sums (even j) or the differences (odd j) of the moments at a
// and n-1-a against half of the nodes; that half of the table is in LDS, a row
// per j, two values a read.  (The whole table, one value a read, and a column
// of 48 moments spilled: 8515 pairs at n = 37 71 us, now 15 us.)
constexpr int kCoefThreads = 256;

template <int NMAX>
__device__ inline void coef_moments_body(const double* __restrict__ M, int n, int64_t npair, int kind,
                                         double* __restrict__ mu) {
  constexpr int H = NMAX / 2;
  __shared__ __align__(16) double V[NMAX * H];   // [j][a < ceil(n / 2)], zero beyond
  const int he = (n + 1) / 2;
  for (int e = threadIdx.x; e < n * H; e += kCoefThreads) {
    const int j = e / H, a = e - j * H;
    V[e] = a < he ? cheb_at_node(kind, n, a, j) : 0.0;
  }
  __syncthreads();
  const int d = blockIdx.y;
  const int64_t p = (int64_t)blockIdx.x * kCoefThreads + threadIdx.x;
  if (p >= npair) return;
  double ms[H], md[H];
#pragma unroll
  for (int a = 0; a < H; ++a) {
    const int b = n - 1 - a;
    const double x = a < he ? M[((int64_t)d * n + a) * npair + p] : 0.0;
    const double y = a < he && b != a ? M[((int64_t)d * n + b) * npair + p] : 0.0;
    ms[a] = x + y;
    md[a] = x - y;   // the middle node: against T_j(0) = 0
  }
  double* out = mu + (int64_t)d * n * npair + p;
#pragma unroll 1
  for (int j = 0; j < n; j += 2) {
    const double* v0 = V + j * H;
    const double* v1 = V + (j + 1 < n ? j + 1 : j) * H;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int a = 0; a < H; ++a) {
      s0 += v0[a] * ms[a];
      s1 += v1[a] * md[a];
      if (a % 4 == 3) __asm__ volatile("" : "+v"(s0), "+v"(s1) : : "memory");   // not both rows in registers
    }
    out[(int64_t)j * npair] = s0;
    if (j + 1 < n) out[(int64_t)(j + 1) * npair] = s1;
  }
}

template <int NMAX>
__global__ void __launch_bounds__(kCoefThreads)
coef_moments_kernel(const double* __restrict__ M, int n, int64_t npair, int kind, double* __restrict__ mu) {
  coef_moments_body<NMAX>(M, n, npair, kind, mu);
}

// blockIdx.z = molecule; molecules without coefficient moments are skipped
template <int NMAX>
__global__ void __launch_bounds__(kCoefThreads)
coef_moments_batch_kernel(const PrepMol* __restrict__ mols, int n, int kind) {
  const PrepMol& m = mols[blockIdx.z];
  if (m.Mu == nullptr || (int64_t)blockIdx.x * kCoefThreads >= m.npair) return;
  coef_moments_body<NMAX>(m.M, n, m.npair, kind, m.Mu);
}

}  // namespace

hipError_t launch_coef_moments(const double* M, int n, int64_t npair, int kind, double* mu, hipStream_t s) {
  const dim3 grid((unsigned)((npair + kCoefThreads - 1) / kCoefThreads), 3);
  if (n <= 16) hipLaunchKernelGGL(coef_moments_kernel<16>, grid, dim3(kCoefThreads), 0, s, M, n, npair, kind, mu);
  else if (n <= 32) hipLaunchKernelGGL(coef_moments_kernel<32>, grid, dim3(kCoefThreads), 0, s, M, n, npair, kind, mu);
  else if (n <= 48) hipLaunchKernelGGL(coef_moments_kernel<48>, grid, dim3(kCoefThreads), 0, s, M, n, npair, kind, mu);
  else hipLaunchKernelGGL(coef_moments_kernel<64>, grid, dim3(kCoefThreads), 0, s, M, n, npair, kind, mu);
  return hipGetLastError();
}

hipError_t launch_coef_moments_batch(const PrepMol* mols, int nmol, int64_t max_npair, int n, int kind,
                                     hipStream_t s) {
  const dim3 grid((unsigned)((max_npair + kCoefThreads - 1) / kCoefThreads), 3, nmol);
  if (n <= 16) hipLaunchKernelGGL(coef_moments_batch_kernel<16>, grid, dim3(kCoefThreads), 0, s, mols, n, kind);
  else if (n <= 32) hipLaunchKernelGGL(coef_moments_batch_kernel<32>, grid, dim3(kCoefThreads), 0, s, mols, n, kind);
  else if (n <= 48) hipLaunchKernelGGL(coef_moments_batch_kernel<48>, grid, dim3(kCoefThreads), 0, s, mols, n, kind);
  else hipLaunchKernelGGL(coef_moments_batch_kernel<64>, grid, dim3(kCoefThreads), 0, s, mols, n, kind);
  return hipGetLastError();
}

// calls f with the compiled inner length for n (2 <= n <= 64) as a constant
template <class F>
static void with_nmax(int n, F f) {
  if (n <= 16) f(std::integral_constant<int, 16>{});
  else if (n <= 24) f(std::integral_constant<int, 24>{});
  else if (n <= 32) f(std::integral_constant<int, 32>{});
  else if (n <= 40) f(std::integral_constant<int, 40>{});
  else if (n <= 48) f(std::integral_constant<int, 48>{});
  else f(std::integral_constant<int, 64>{});
}
static unsigned moment_blocks(int64_t npair) { return (unsigned)((3 * npair + kMomThreads - 1) / kMomThreads); }

hipError_t launch_moments_batch(const PrepMol* mols, int nmol, int64_t max_npair, int n, hipStream_t s) {
  const dim3 grid(moment_blocks(max_npair), nmol);
  with_nmax(n, [&](auto c) {
    hipLaunchKernelGGL(moments_batch_kernel<decltype(c)::value>, grid, dim3(kMomThreads), 0, s, mols, n);
  });
  return hipGetLastError();
}

hipError_t launch_moments_pairs(const DevBasis& b, int n, double L, const NodeTables& tb, const int32_t* pairs,
                                int64_t npair, double* M, hipStream_t s) {
  with_nmax(n, [&](auto c) {
    hipLaunchKernelGGL(moments_kernel<decltype(c)::value>, dim3(moment_blocks(npair)), dim3(kMomThreads), 0, s, b, n,
                       L, tb, M, npair, pairs);
  });
  return hipGetLastError();
}

hipError_t launch_moments_parts(const DevBasis& b, int n, const NodeTables& tb, const int32_t* pairs,
                                const PartSpans& sp, int nparts, double* M, hipStream_t s) {
  int64_t maxc = 0;
  for (int z = 0; z < nparts; ++z) maxc = std::max<int64_t>(maxc, sp.off[z + 1] - sp.off[z]);
  if (maxc == 0) return hipSuccess;
  const dim3 grid(moment_blocks(maxc), (unsigned)nparts);
  with_nmax(n, [&](auto c) {
    hipLaunchKernelGGL(moments_parts_kernel<decltype(c)::value>, grid, dim3(kMomThreads), 0, s, b, n, sp, tb, M, pairs);
  });
  return hipGetLastError();
}

hipError_t launch_moments(const DevBasis& b, int n, double L, const NodeTables& tb,
                          double* M, hipStream_t s) {
  return launch_moments_pairs(b, n, L, tb, nullptr, (int64_t)b.nb * (b.nb + 1) / 2, M, s);
}

hipError_t launch_screen(const DevBasis& b, double tau, int32_t* rows, int32_t* pairs, int32_t* count,
                         hipStream_t s) {
  const unsigned blocks = (unsigned)((b.nb + kScreenRows - 1) / kScreenRows);
  hipLaunchKernelGGL(screen_count_kernel, dim3(blocks), dim3(kScreenThreads), 0, s, b, tau, rows);
  hipLaunchKernelGGL(screen_scan_kernel, dim3(1), dim3(1024), 0, s, b.nb, rows, count);
  hipLaunchKernelGGL(screen_write_kernel, dim3(blocks), dim3(kScreenThreads), 0, s, b, tau, rows, pairs);
  return hipGetLastError();
}

}  // namespace tai
