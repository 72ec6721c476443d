// Quadrature and interpolation tables on the device, FP64.
//
// * Gauss-Legendre nodes/weights for int_0^omega ds (eq. TEI2 with the
//   Gauss rule of Prop. 2.4), by Newton's method on the Legendre polynomial.
// * Chebyshev nodes on [-L, L], Lobatto or first kind (Def. 2.2).
// * K_k(a,b) = exp(-t_k^2 (xi_a - xi_b)^2): the 1D Gaussian factor of
//   eq. TEI2 on the Chebyshev grid, i.e. the node-value form of the
//   interpolant of eq. chebcheb.
// * The map from Chebyshev moments to Lagrange moments used by the moment
//   kernel: l_a(x) = sum_k gam[a][k] T_k(x/L).
// * Per-node degrees (eq. chebcheb with N_k points for node k): the Chebyshev
//   coefficients of each node's factor, the smallest degree whose dropped
//   coefficients sum to at most a tolerance, and the truncated K tables.
#include "tai_internal.h"
#include "tai_device.h"

#include <cmath>

namespace tai {
namespace {

constexpr int kNodeThreads = 256;
constexpr int kMaxNodes = 128, kMaxGrid = 64;
// entries of one K_k that a work group fills: four exponentials per thread
constexpr int kNodeEntries = 4 * kNodeThreads;

// Entries of gam written: the n*n map and zeros up to its 256-byte boundary,
// so that the moment kernel may read whole padded rows.
__host__ __device__ inline int64_t gam_entries(int n) { return ((int64_t)n * n + 31) / 32 * 32; }

// Root `i` (0-based, descending) of P_m and its Gauss weight, by Newton's method
// on the three-term recurrence P_{j+1} = a_j x P_j - b_j P_{j-1} (ab[j] = (a_j,
// b_j): one dependent operation a step).  The start value is cos of the
// asymptotic angle with its first correction, good to about m^-4, so that the
// third step is below rounding; the last evaluation then also gives P_m' for the
// weight.
__device__ inline void gauss_root(int m, int i, const double2* ab, double& x, double& wt) {
  x = (1.0 - (m - 1.0) / (8.0 * m * m * m)) * cos(M_PI * (i + 0.75) / (m + 0.5));
  double dp = 1.0;
  for (int it = 0; it < 100; ++it) {
    double p0 = 1.0, p1 = x;
#pragma unroll 4
    for (int j = 1; j < m; ++j) {
      const double2 c = ab[j];
      const double p2 = fma(c.x * x, p1, -(c.y * p0));
      p0 = p1;
      p1 = p2;
    }
    dp = m * (x * p1 - p0) / (x * x - 1.0);
    const double dx = p1 / dp;
    x -= dx;
    if (fabs(dx) < 1e-15) break;
  }
  wt = 2.0 / ((1.0 - x * x) * dp * dp);
}

// Work groups of the tables that `parts` names: nq node groups (times the pieces
// of a K table), then those of gam.
__host__ __device__ inline int node_pieces(int n, unsigned parts) {
  return parts & kTablesK ? (n * n + kNodeEntries - 1) / kNodeEntries : 1;
}
__host__ __device__ inline int node_groups(int nq, int n, unsigned parts) {
  return parts & (kTablesK | kTablesNodes) ? nq * node_pieces(n, parts) : 0;
}
inline int table_groups(int nq, int n, unsigned parts) {
  return node_groups(nq, n, parts) +
         (parts & kTablesGam ? (int)((gam_entries(n) + kNodeThreads - 1) / kNodeThreads) : 0);
}

// One launch: a work group of a K_k works out its own node t_k (and one of them
// writes it), others fill the map gam.
//   What bounds it: latency, the recurrence's chain.  With the nodes in a launch of
// their own, a division in every step and six evaluations: 24 nodes at n = 32
// 12.5 us for the two launches, now 6.8 us (the moments, which read gam alone, 1.5).
__device__ inline void tables_body(double omega, int nq, int n, double L, int kind, unsigned parts,
                                   const NodeTables& tb) {
  __shared__ double2 ab[kMaxNodes];
  __shared__ double s_xi[kMaxGrid];
  __shared__ double s_t;
  const int tid = threadIdx.x, ng = node_groups(nq, n, parts);
  if ((int)blockIdx.x < ng) {
    const int pieces = node_pieces(n, parts);
    const int k = blockIdx.x / pieces, piece = blockIdx.x % pieces;
    if (tid >= 128) {
      const int j = tid - 128;
      if (j > 0 && j < nq) ab[j] = double2{(2.0 * j + 1.0) / (j + 1.0), j / (j + 1.0)};
    } else if (tid >= 64 && tid - 64 < n) {
      const int a = tid - 64;
      const double th = (kind == 0) ? M_PI * a / (n - 1) : (2.0 * a + 1.0) * M_PI / (2.0 * n);
      const double xi = L * cos(th);
      s_xi[a] = xi;
      if (blockIdx.x == 0) tb.xi[a] = xi;
    }
    __syncthreads();
    if (tid < 64) {
      double z, zw;
      gauss_root(nq, nq - 1 - k, ab, z, zw);  // ascending order
      if (tid == 0) {
        const double t = 0.5 * omega * (1.0 + z);
        s_t = t;
        if (piece == 0) {
          tb.t[k] = t;
          tb.w[k] = 0.5 * omega * zw;
        }
      }
    }
    if (!(parts & kTablesK)) return;
    __syncthreads();
    const double t = s_t;
    double* Kk = tb.K + (int64_t)k * n * n;
#pragma unroll
    for (int r = 0; r < kNodeEntries / kNodeThreads; ++r) {
      const int e = piece * kNodeEntries + r * kNodeThreads + tid;
      if (e < n * n) {
        const double dx = s_xi[e / n] - s_xi[e % n];
        Kk[e] = exp(-t * t * dx * dx);
      }
    }
    return;
  }
  const int ak = ((int)blockIdx.x - ng) * kNodeThreads + tid;
  if (ak >= gam_entries(n)) return;
  const int a = ak / n, k = ak % n;
  double v;
  if (ak >= n * n) {
    v = 0.0;
  } else if (kind == 0) {
    // Lobatto: l_a(u) = sum_k 2/(N c_a c_k) T_k(u_a) T_k(u), N = n-1,
    // c_0 = c_N = 2, other c = 1; T_k(u_a) = cos(pi a k / N)
    const int N = n - 1;
    const double ca = (a == 0 || a == N) ? 2.0 : 1.0;
    const double ck = (k == 0 || k == N) ? 2.0 : 1.0;
    v = 2.0 / (N * ca * ck) * cos(M_PI * (double)((int64_t)a * k % (2 * N)) / N);
  } else {
    // first kind: l_a(u) = sum_k (2 - delta_k0)/n T_k(u_a) T_k(u),
    // T_k(u_a) = cos(k (2a+1) pi / (2n))
    const double ck = (k == 0) ? 1.0 : 2.0;
    v = ck / n * cos(M_PI * (double)((int64_t)k * (2 * a + 1) % (4 * n)) / (2.0 * n));
  }
  tb.gam[ak] = v;
}

__global__ void __launch_bounds__(kNodeThreads)
tables_kernel(double omega, int nq, int n, double L, int kind, unsigned parts, NodeTables tb) {
  tables_body(omega, nq, n, L, kind, parts, tb);
}

// molecule blockIdx.y
__global__ void __launch_bounds__(kNodeThreads)
tables_batch_kernel(const PrepMol* __restrict__ mols, int nq, int n, int kind) {
  const PrepMol& m = mols[blockIdx.y];
  tables_body(m.omega, nq, n, m.L, kind, kTablesAll, m.tb);
}

constexpr int kDegThreads = 1024;
constexpr int kDegMaxN = 64;
constexpr int kDegPer = kDegMaxN * kDegMaxN / kDegThreads;  // entries per thread

// One work group per node k.  With gam the Chebyshev-to-Lagrange map
// (l_a = sum_j gam[a][j] T_j), the node's interpolant
// sum_ab K_k(a,b) l_a(x) l_b(y) has coefficients C = gam^T K_k gam.  The
// coefficients are summed in absolute value over the shells max(i,j) = s,
// and the tail sums tail(m) = sum_{s >= m} shell(s) taken from the outside
// in: N_k is the smallest m >= 1 with tail(m) <= tol (n if tol <= 0).
// Dropping the rest moves the factor by at most tail(N_k) on the box since
// |T_j| <= 1.  With tol > 0, K_k becomes V C V^T, V[a][j] = T_j(xi_a/L): the
// node values of the kept polynomial, which every node-form stage uses.
//   What bounds it: latency, nq work groups of four n x n products.  Both
// factors come from LDS and V is a table there: from memory, with a cosine in
// the inner loop, n = 37 took 206 us, now 18 us.
__device__ inline void degrees_body(int n, int kind, double tol, const NodeTables& tb, int k) {
  __shared__ double s_a[kDegMaxN * kDegMaxN], s_b[kDegMaxN * kDegMaxN], s_g[kDegMaxN * kDegMaxN];
  __shared__ double shell[kDegMaxN];
  __shared__ int nk_s;
  const int tid = threadIdx.x, nn = n * n;
  const double* Kk = tb.K + (int64_t)k * nn;
  // out = sum over c < len of f(row, c) g(c, col) for every entry
  auto product = [&](double* out, int len, auto f, auto g) {
#pragma unroll
    for (int r = 0; r < kDegPer; ++r) {
      const int e = tid + kDegThreads * r;
      if (e < nn) {
        const int i = e / n, j = e - i * n;
        double x = 0.0;
        for (int c = 0; c < len; ++c) x += f(i, c) * g(c, j);
        out[e] = x;
      }
    }
    __syncthreads();
  };
  for (int e = tid; e < nn; e += kDegThreads) {
    s_a[e] = Kk[e];
    s_g[e] = tb.gam[e];
  }
  __syncthreads();
  product(s_b, n, [&](int a, int b) { return s_a[a * n + b]; }, [&](int b, int j) { return s_g[b * n + j]; });
  product(s_a, n, [&](int i, int a) { return s_g[a * n + i]; }, [&](int a, int j) { return s_b[a * n + j]; });
  // s_a = C; V into s_g
  for (int e = tid; e < nn; e += kDegThreads) s_g[e] = cheb_at_node(kind, n, e / n, e % n);
  if (tid < n) {
    const int s = tid;
    double x = 0.0;
    for (int j = 0; j <= s; ++j) x += fabs(s_a[s * n + j]);
    for (int i = 0; i < s; ++i) x += fabs(s_a[i * n + s]);
    shell[s] = x;
  }
  __syncthreads();
  if (tid == 0) {
    int m = n;
    if (tol > 0) {
      double tail = 0.0;
      for (int c = n - 1; c >= 1; --c) {
        tail += shell[c];
        if (tail <= tol) m = c;
        else break;
      }
    }
    nk_s = m;
    tb.nk[k] = m;
  }
  __syncthreads();
  const int m = nk_s;
  double* Ck = tb.C + (int64_t)k * nn;
  for (int e = tid; e < nn; e += kDegThreads) {
    const int i = e / n, j = e - i * n;
    const double c = (i < m && j < m) ? s_a[e] : 0.0;
    Ck[e] = c;
    s_a[e] = c;
  }
  if (!(tol > 0)) return;
  __syncthreads();
  // Z = C V^T, then K~ = V Z
  product(s_b, m, [&](int i, int j) { return s_a[i * n + j]; }, [&](int j, int b) { return s_g[b * n + j]; });
  double* Kw = tb.K + (int64_t)k * nn;
#pragma unroll
  for (int r = 0; r < kDegPer; ++r) {
    const int e = tid + kDegThreads * r;
    if (e < nn) {
      const int a = e / n, b = e - a * n;
      double x = 0.0;
      for (int i = 0; i < m; ++i) x += s_g[a * n + i] * s_b[i * n + b];
      Kw[e] = x;
    }
  }
}

__global__ void __launch_bounds__(kDegThreads)
degrees_kernel(int n, int kind, double tol, NodeTables tb) {
  degrees_body(n, kind, tol, tb, blockIdx.x);
}

// one work group per (node, molecule); molecules with tol <= 0 are skipped
__global__ void __launch_bounds__(kDegThreads)
degrees_batch_kernel(const PrepMol* __restrict__ mols, int n, int kind) {
  const PrepMol& m = mols[blockIdx.y];
  if (!(m.degree_tol > 0)) return;
  degrees_body(n, kind, m.degree_tol, m.tb, blockIdx.x);
}

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

}  // namespace

size_t node_tables_bytes(int nq, int n) {
  return align256(sizeof(double) * nq) * 2 + align256(sizeof(double) * n) +
         align256(sizeof(double) * (size_t)nq * n * n) + align256(sizeof(double) * n * n) +
         align256(sizeof(double) * (size_t)nq * n * n) + align256(sizeof(int32_t) * nq);
}

NodeTables carve_node_tables(void* base, int nq, int n) {
  char* p = static_cast<char*>(base);
  NodeTables tb;
  tb.t = reinterpret_cast<double*>(p); p += align256(sizeof(double) * nq);
  tb.w = reinterpret_cast<double*>(p); p += align256(sizeof(double) * nq);
  tb.xi = reinterpret_cast<double*>(p); p += align256(sizeof(double) * n);
  tb.K = reinterpret_cast<double*>(p); p += align256(sizeof(double) * (size_t)nq * n * n);
  tb.gam = reinterpret_cast<double*>(p); p += align256(sizeof(double) * n * n);
  tb.C = reinterpret_cast<double*>(p); p += align256(sizeof(double) * (size_t)nq * n * n);
  tb.nk = reinterpret_cast<int32_t*>(p);
  return tb;
}

hipError_t launch_degrees(int nq, int n, int kind, double degree_tol, const NodeTables& tb, hipStream_t s) {
  if (n > kDegMaxN) return hipErrorInvalidValue;
  hipLaunchKernelGGL(degrees_kernel, dim3(nq), dim3(kDegThreads), 0, s, n, kind, degree_tol, tb);
  return hipGetLastError();
}

hipError_t launch_nodes(double omega, int nq, int n, double L, int kind, double degree_tol,
                        const NodeTables& tb, hipStream_t s, unsigned parts) {
  if (nq > kMaxNodes || n > kMaxGrid) return hipErrorInvalidValue;
  if (degree_tol > 0) parts = kTablesAll;
  hipLaunchKernelGGL(tables_kernel, dim3(table_groups(nq, n, parts)), dim3(kNodeThreads), 0, s, omega, nq, n, L, kind,
                     parts, tb);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !(degree_tol > 0)) return e;
  return launch_degrees(nq, n, kind, degree_tol, tb, s);
}

hipError_t launch_nodes_batch(const PrepMol* mols, int nmol, int nq, int n, int kind, bool any_degree,
                              hipStream_t s) {
  if (nq > kMaxNodes || n > kMaxGrid) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tables_batch_kernel, dim3(table_groups(nq, n, kTablesAll), nmol), dim3(kNodeThreads), 0, s, mols,
                     nq, n, kind);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !any_degree) return e;
  if (n > kDegMaxN) return hipErrorInvalidValue;
  hipLaunchKernelGGL(degrees_batch_kernel, dim3(nq, nmol), dim3(kDegThreads), 0, s, mols, n, kind);
  return hipGetLastError();
}

}  // namespace tai
