// Polynomial chaos by stochastic collocation (section 3, Eq. 27-28).
//
// The expansion w(x, xi) ~ sum_i w_i(x) Psi_i(xi) uses products of
// one-dimensional polynomials orthonormal under each input's distribution
// (probabilists' Hermite for a standard normal input, Legendre for a uniform
// input on [-1, 1]) over every multi-index of total degree <= p.  Its
// coefficients come from the least-squares solution of the Vandermonde
// system V W = Y at M sample points (Eq. 28), for every output x at once.
//
// Host side (sizes of a few hundred): Gauss rules, tensor and Smolyak node
// sets, the basis and V.  Device side: W = P Y, the evaluation V_test W at test
// points, and the per-output mean, variance and Sobol indices.  The projection P
// = R^-1 Q^T of a Householder QR of V is formed on the host for small sets and on
// the device otherwise (host_projection).
#include "common.h"

#include <algorithm>
#include <cmath>
#include <functional>
#include <map>

struct ppe_pce {
  int d = 0, degree = 0, n_terms = 0;
  std::vector<int> kinds;   // PPE_INPUT_NORMAL / PPE_INPUT_UNIFORM per input
  std::vector<int> alpha;   // n_terms x d multi-indices, graded order
  hipStream_t stream = nullptr;
  int device = 0;
  std::string err;
  ppe::DevBuf a_dev, mask_dev, qr_dev;
  size_t lds_max = 0;    // LDS one workgroup may use (0: not queried yet)
  int* bad_h = nullptr;  // pinned: whether the last fit's points were rank deficient
  ~ppe_pce() {
    if (bad_h) (void)hipHostFree(bad_h);
  }
};

namespace ppe {
namespace {

// orthonormal recurrence x psi_k = b_{k+1} psi_{k+1} + b_k psi_{k-1} (zero
// diagonal for both symmetric families): Hermite b_k = sqrt(k), Legendre
// b_k = k / sqrt(4k^2 - 1)
double rec_b(int kind, int k) {
  if (k == 0) return 0.0;  // multiplies psi_{-1} = 0
  return kind == PPE_INPUT_NORMAL ? std::sqrt((double)k) : k / std::sqrt(4.0 * k * k - 1.0);
}

// psi_0..psi_n at x; returns psi_n, and psi_{n-1} in *prev
double psi_n(int kind, int n, double x, double* prev) {
  double pm = 0.0, p = 1.0;
  for (int k = 0; k < n; ++k) {
    const double next = (x * p - rec_b(kind, k) * pm) / rec_b(kind, k + 1);
    pm = p;
    p = next;
  }
  if (prev) *prev = pm;
  return p;
}

// n-point Gauss rule with probability weights: roots of psi_n found between
// consecutive roots of psi_{n-1} (interlacing) by bisection, polished by
// Newton; weights from the Christoffel numbers 1 / sum_{k<n} psi_k(x)^2.
void gauss_rule(int kind, int n, std::vector<double>& x, std::vector<double>& w) {
  std::vector<double> prev_roots;
  const double outer = kind == PPE_INPUT_NORMAL ? std::sqrt(4.0 * n + 2.0) + 1.0 : 1.0;
  std::vector<double> roots;
  for (int m = 1; m <= n; ++m) {
    roots.assign(m, 0.0);
    for (int i = 0; i < m; ++i) {
      double lo = i == 0 ? -outer : prev_roots[i - 1];
      double hi = i == m - 1 ? outer : prev_roots[i];
      double flo = psi_n(kind, m, lo, nullptr);
      for (int it = 0; it < 200 && hi - lo > 1e-16 * std::max(1.0, std::fabs(lo)); ++it) {
        const double mid = 0.5 * (lo + hi);
        const double fm = psi_n(kind, m, mid, nullptr);
        if ((fm < 0) == (flo < 0)) {
          lo = mid;
          flo = fm;
        } else {
          hi = mid;
        }
      }
      roots[i] = 0.5 * (lo + hi);
    }
    prev_roots = roots;
  }
  x.assign(n, 0.0);
  w.assign(n, 0.0);
  for (int i = 0; i < n; ++i) {
    double r = roots[i];
    for (int it = 0; it < 3; ++it) {  // Newton, psi_n' from the differentiated recurrence
      double pm = 0.0, p = 1.0, dpm = 0.0, dp = 0.0;
      for (int k = 0; k < n; ++k) {
        const double b1 = rec_b(kind, k + 1), b0 = rec_b(kind, k);
        const double next = (r * p - b0 * pm) / b1;
        const double dnext = (p + r * dp - b0 * dpm) / b1;
        pm = p;
        p = next;
        dpm = dp;
        dp = dnext;
      }
      if (dp == 0.0) break;
      r -= p / dp;
    }
    x[i] = r;
  }
  // exact symmetry about 0
  for (int i = 0; i < n / 2; ++i) {
    const double s = 0.5 * (x[n - 1 - i] - x[i]);
    x[i] = -s;
    x[n - 1 - i] = s;
  }
  if (n % 2) x[n / 2] = 0.0;
  for (int i = 0; i < n; ++i) {
    double pm = 0.0, p = 1.0, s = 1.0;
    for (int k = 0; k + 1 < n; ++k) {
      const double next = (x[i] * p - rec_b(kind, k) * pm) / rec_b(kind, k + 1);
      pm = p;
      p = next;
      s += p * p;
    }
    w[i] = 1.0 / s;
  }
}

struct NodeSet {
  std::map<std::vector<long long>, std::pair<std::vector<double>, double>> pts;
  void add(const std::vector<double>& x, double w) {
    std::vector<long long> key(x.size());
    for (size_t j = 0; j < x.size(); ++j) key[j] = std::llround(x[j] * 1e12);  // identifies coincident nodes
    auto it = pts.find(key);
    if (it == pts.end()) pts.emplace(key, std::make_pair(x, w));
    else it->second.second += w;
  }
};

long long binom(int n, int k) {
  if (k < 0 || k > n) return 0;
  long long r = 1;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

void add_tensor(NodeSet& S, const std::vector<int>& kinds, const std::vector<int>& npts, double coef) {
  const int d = (int)kinds.size();
  std::vector<std::vector<double>> xs(d), ws(d);
  for (int j = 0; j < d; ++j) gauss_rule(kinds[j], npts[j], xs[j], ws[j]);
  std::vector<int> c(d, 0);
  std::vector<double> x(d);
  for (;;) {
    double w = coef;
    for (int j = 0; j < d; ++j) {
      x[j] = xs[j][c[j]];
      w *= ws[j][c[j]];
    }
    S.add(x, w);
    int j = 0;
    while (j < d && ++c[j] == npts[j]) c[j++] = 0;
    if (j == d) break;
  }
}

// P = R^-1 Q^T (K rows of ldp) of V (M x K, row-major) by Householder QR on the
// host, which takes small sets (host_projection).  Returns false, P unwritten,
// if a column's remainder's norm is at most `tiny`.
bool projection_host(int M, int K, const double* V, double tiny, double* P, int ldp) {
  // rows are points, so that a reflection runs along contiguous columns
  std::vector<double> A(V, V + (size_t)M * K), Q((size_t)M * K, 0.0), v((size_t)K * M), c(K), s(K);
  for (int k = 0; k < K; ++k) {
    double* vk = v.data() + (size_t)k * M;
    double nn = 0.0;
    for (int i = k; i < M; ++i) nn += A[(size_t)i * K + k] * A[(size_t)i * K + k];
    const double nrm = std::sqrt(nn), akk = A[(size_t)k * K + k];
    if (!(nrm > tiny)) return false;
    for (int i = k; i < M; ++i) vk[i] = A[(size_t)i * K + k];
    vk[k] -= akk > 0 ? -nrm : nrm;
    c[k] = 1.0 / (nn + std::fabs(akk) * nrm);  // 2 / (v . v)
    std::fill(s.begin() + k, s.end(), 0.0);
    for (int i = k; i < M; ++i)
      for (int j = k; j < K; ++j) s[j] += vk[i] * A[(size_t)i * K + j];
    for (int i = k; i < M; ++i)
      for (int j = k; j < K; ++j) A[(size_t)i * K + j] -= c[k] * s[j] * vk[i];
  }
  // Q's columns: the reflections of the identity's, last to first
  for (int k = K - 1; k >= 0; --k) {
    const double* vk = v.data() + (size_t)k * M;
    Q[(size_t)k * K + k] = 1.0;
    std::fill(s.begin() + k, s.end(), 0.0);
    for (int i = k; i < M; ++i)
      for (int j = k; j < K; ++j) s[j] += vk[i] * Q[(size_t)i * K + j];
    for (int i = k; i < M; ++i)
      for (int j = k; j < K; ++j) Q[(size_t)i * K + j] -= c[k] * s[j] * vk[i];
  }
  // R P = Q^T, all points at once
  for (int i = K - 1; i >= 0; --i) {
    double* p = P + (size_t)i * ldp;
    for (int m = 0; m < M; ++m) p[m] = Q[(size_t)m * K + i];
    for (int j = i + 1; j < K; ++j) {
      const double r = A[(size_t)i * K + j], *pj = P + (size_t)j * ldp;
      for (int m = 0; m < M; ++m) p[m] -= r * pj[m];
    }
    for (int m = 0; m < M; ++m) p[m] /= A[(size_t)i * K + i];
  }
  return true;
}

// ---- P = R^-1 Q^T on the device.  A fit at the paper's sizes (216 points, 56
// terms) is a serial chain of K reflections of a matrix that one compute unit
// holds, so one workgroup takes it all.  Up to 256 points and 64 terms
// (k_projection_regs) every wave keeps every 16th column in registers: the
// wave of column k forms its reflector and leaves it in LDS, and one barrier
// later every wave reflects its own columns.  Q's first K columns come from
// the reflectors, last to first, without a barrier, and four lanes per point
// solve R p = q.  What is left is the chain itself: a reduction over the
// wave, a barrier, a dot product and its reduction, K times.  216 x 56: 138
// us; with the columns in LDS 481, and 1.7 ms on the host, where Q^T had been
// accumulated on the whole identity.  Larger sets run k_projection, columns
// in global memory (a reflection's columns then come from L2 each step).
constexpr int kQrThreads = 1024, kQrWaves = kQrThreads / kWave;
constexpr int kQrRows = 4, kQrCols = 4;  // registers: rows per lane, columns per wave

// v moved by a DPP pattern (lanes without a source get 0).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
  const long long x = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, ROWS, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double read_lane(double v, int lane) {
  const long long x = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)x, lane);
  const int hi = __builtin_amdgcn_readlane((int)(x >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the wave, the same in every lane: row sums (shifts by 1, 2, 4 and 8
// within rows of 16), then across the rows; no LDS.
__device__ __forceinline__ double wave_all_sum(double v) {
  v += dpp_move<0x111, 0xf>(v);
  v += dpp_move<0x112, 0xf>(v);
  v += dpp_move<0x114, 0xf>(v);
  v += dpp_move<0x118, 0xf>(v);
  v += dpp_move<0x142, 0xa>(v);  // the row below's last lane into rows 1 and 3
  v += dpp_move<0x143, 0xc>(v);  // lane 31 into rows 2 and 3
  return read_lane(v, kWave - 1);
}

// The upper half's v of x exchanged with the lower half's of y (HALF lanes of
// every 2 HALF, HALF 32 or 16), then added: in the lower lanes the pair sums
// of x, in the upper ones those of y.
template <int HALF>
__device__ __forceinline__ double swap_add(double x, double y) {
  const long long a = __builtin_bit_cast(long long, x), b = __builtin_bit_cast(long long, y);
  double u, v;
  if constexpr (HALF == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap((int)a, (int)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((int)(a >> 32), (int)(b >> 32), false, false);
    u = __builtin_bit_cast(double, ((long long)hi[0] << 32) | (unsigned int)lo[0]);
    v = __builtin_bit_cast(double, ((long long)hi[1] << 32) | (unsigned int)lo[1]);
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap((int)a, (int)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((int)(a >> 32), (int)(b >> 32), false, false);
    u = __builtin_bit_cast(double, ((long long)hi[0] << 32) | (unsigned int)lo[0]);
    v = __builtin_bit_cast(double, ((long long)hi[1] << 32) | (unsigned int)lo[1]);
  }
  return u + v;
}

// Four sums over the wave at once, each then in every lane: the halves and
// rows are exchanged so that one value per lane is left after two steps (row
// q of 16 lanes holds the q-th of d0, d2, d1, d3), a third of the
// instructions of four wave_all_sum.
__device__ __forceinline__ void wave_all_sum4(double (&d)[4]) {
  double v = swap_add<16>(swap_add<32>(d[0], d[1]), swap_add<32>(d[2], d[3]));
  v += dpp_move<0x111, 0xf>(v);
  v += dpp_move<0x112, 0xf>(v);
  v += dpp_move<0x114, 0xf>(v);
  v += dpp_move<0x118, 0xf>(v);
  d[0] = read_lane(v, 15);
  d[2] = read_lane(v, 31);
  d[1] = read_lane(v, 47);
  d[3] = read_lane(v, 63);
}

// Small sets are factorised on the host: it needs no dispatch and no upload of V,
// and a reflection costs it 4 M K / 10^4 us where the device's chain takes 2.5 and
// the dispatches 15 more.  Fits of 1,000 outputs, host and device: 2 x 2 20 and 33
// us, 10 x 10 23 and 52, 60 x 20 39 and 82, 105 x 35 99 and 132, 84 x 56 136 and
// 175; the two meet near 4,000 + 40 K values: 200 x 20 94 and 105, 168 x 28 118 and
// 123, 210 x 35 186 and 155, 123 x 56 201 and 185.
inline bool host_projection(int M, int K) { return (int64_t)M * K < 4000 + 40 * (int64_t)K; }

// A workspace of a factorisation: the columns, R (K x K) and 2 / (v . v).
inline size_t qr_words(int M, int K) { return (size_t)K * M + (size_t)K * K + K; }

// V: M x K row-major.  A column whose remainder's norm is at most `tiny`
// (rank deficiency) sets *bad, and P (K rows of ldp) stays unwritten; *bad is
// 0 otherwise.  M <= 64 kQrRows, K <= 16 kQrCols, qr_words(M, K) doubles of LDS.
__global__ void __launch_bounds__(kQrThreads) k_projection_regs(int M, int K,
                                                                const double* __restrict__ V,
                                                                double tiny,
                                                                double* __restrict__ P, int ldp,
                                                                int* __restrict__ bad,
                                                                int* __restrict__ bad_host) {
  extern __shared__ double qr_lds[];
  __shared__ int stop;
  double* S = qr_lds;             // reflector k at S + k M, then Q's columns
  double* R = S + (size_t)K * M;  // K x K, row-major, upper triangle
  double* vv = R + (size_t)K * K;
  const int t = threadIdx.x, lane = t % kWave;
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  if (t == 0) stop = 0;
  double a[kQrCols][kQrRows];
#pragma unroll
  for (int c = 0; c < kQrCols; ++c)
#pragma unroll
    for (int r = 0; r < kQrRows; ++r) {
      const int j = w + c * kQrWaves, row = lane + r * kWave;
      a[c][r] = j < K && row < M ? V[row * K + j] : 0.0;
    }
  for (int k = 0; k < K; ++k) {
    if (w == k % kQrWaves) {
      double x[kQrRows], s = 0.0, own = 0.0;
#pragma unroll
      for (int r = 0; r < kQrRows; ++r) {
        x[r] = 0.0;
#pragma unroll
        for (int c = 0; c < kQrCols; ++c)
          if (c == k / kQrWaves) x[r] = a[c][r];
        if (lane + r * kWave >= k) s = fma(x[r], x[r], s);
        if (r == k / kWave) own = x[r];
      }
      s = wave_all_sum(s);
      const double nrm = sqrt(s), vk = read_lane(own, k % kWave);
      const double alpha = vk > 0 ? -nrm : nrm;
#pragma unroll
      for (int r = 0; r < kQrRows; ++r) {
        const int row = lane + r * kWave;
        if (row < M) S[k * M + row] = row < k ? 0.0 : row == k ? vk - alpha : x[r];
      }
      if (lane == 0) {
        if (!(nrm > tiny)) stop = 1;
        R[k * K + k] = alpha;
        vv[k] = 1.0 / (s + fabs(vk) * nrm);  // v.v = 2 (s + |v_k| nrm): no cancellation
      }
    }
    __syncthreads();
    if (stop) {
      if (t == 0) *bad = *bad_host = 1;
      return;
    }
    if (w + (kQrCols - 1) * kQrWaves <= k) continue;  // no column past k
    double v[kQrRows], dot[kQrCols];
#pragma unroll
    for (int r = 0; r < kQrRows; ++r) {
      const int row = lane + r * kWave;
      v[r] = row < M ? S[k * M + row] : 0.0;
    }
    const double c2 = vv[k];
#pragma unroll
    for (int c = 0; c < kQrCols; ++c) {
      dot[c] = 0.0;
      if (w + c * kQrWaves <= k) continue;  // reflected already
#pragma unroll
      for (int r = 0; r < kQrRows; ++r) dot[c] = fma(v[r], a[c][r], dot[c]);
    }
    wave_all_sum4(dot);
#pragma unroll
    for (int c = 0; c < kQrCols; ++c) {
      const int j = w + c * kQrWaves;
      if (j <= k) continue;
      const double f = -c2 * dot[c];
#pragma unroll
      for (int r = 0; r < kQrRows; ++r) {
        a[c][r] = fma(f, v[r], a[c][r]);
        if (lane + r * kWave == k && j < K) R[k * K + j] = a[c][r];
      }
    }
  }
  // Q's columns: the reflections of the identity's, last to first (column j
  // is untouched by those past it)
#pragma unroll
  for (int c = 0; c < kQrCols; ++c)
#pragma unroll
    for (int r = 0; r < kQrRows; ++r)
      a[c][r] = w + c * kQrWaves == lane + r * kWave ? 1.0 : 0.0;
  for (int k = K - 1; k >= 0; --k) {
    double v[kQrRows], dot[kQrCols];
#pragma unroll
    for (int r = 0; r < kQrRows; ++r) {
      const int row = lane + r * kWave;
      v[r] = row < M ? S[k * M + row] : 0.0;
    }
    const double c2 = vv[k];
#pragma unroll
    for (int c = 0; c < kQrCols; ++c) {
      dot[c] = 0.0;
      if (w + c * kQrWaves < k) continue;  // still the identity's past row k
#pragma unroll
      for (int r = 0; r < kQrRows; ++r) dot[c] = fma(v[r], a[c][r], dot[c]);
    }
    wave_all_sum4(dot);
#pragma unroll
    for (int c = 0; c < kQrCols; ++c) {
      if (w + c * kQrWaves < k) continue;
      const double f = -c2 * dot[c];
#pragma unroll
      for (int r = 0; r < kQrRows; ++r) a[c][r] = fma(f, v[r], a[c][r]);
    }
  }
  __syncthreads();  // every wave is done with the reflectors
#pragma unroll
  for (int c = 0; c < kQrCols; ++c)
#pragma unroll
    for (int r = 0; r < kQrRows; ++r) {
      const int j = w + c * kQrWaves, row = lane + r * kWave;
      if (j < K && row < M) S[j * M + row] = a[c][r];
    }
  __syncthreads();
  // R p = q for point m: lane g of the four holds p_j, j = g mod 4
  const int m = t / 4, g = t % 4;
  double p[kQrCols * kQrWaves / 4];
#pragma unroll
  for (int q = 0; q < kQrCols * kQrWaves / 4; ++q) p[q] = 0.0;
#pragma unroll
  for (int q = kQrCols * kQrWaves / 4 - 1; q >= 0; --q)
#pragma unroll
    for (int h = 3; h >= 0; --h) {
      const int i = 4 * q + h;
      if (i >= K) continue;
      double x = 0.0, y = 0.0;
#pragma unroll
      for (int u = q; u < kQrCols * kQrWaves / 4; ++u) {
        const int j = 4 * u + g;
        const double rij = j > i && j < K ? R[i * K + j] : 0.0;
        if (u & 1)
          y = fma(rij, p[u], y);
        else
          x = fma(rij, p[u], x);
      }
      x += y;
      x += dpp_move<0xB1, 0xf>(x);  // lanes 1 0 3 2
      x += dpp_move<0x4E, 0xf>(x);  // lanes 2 3 0 1
      const double pi = m < M ? (S[i * M + m] - x) / R[i * K + i] : 0.0;
      if (g == h) {
        p[q] = pi;
        if (m < M) P[i * ldp + m] = pi;
      }
    }
  if (t == 0) *bad = *bad_host = 0;
}

// Columns j = j0, j0 + 16, ... < K of A (M rows each) reflected by v (entries
// below k0 zero): a -= c (v . a) v.  One wave.
__device__ __forceinline__ void reflect(int M, int K, int j0, int k0, double c,
                                        const double* __restrict__ v, double* __restrict__ A) {
  const int lane = threadIdx.x % kWave;
  for (; j0 < K; j0 += 4 * kQrWaves) {
    double dot[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r = (k0 & ~(kWave - 1)) + lane; r < M; r += kWave) {
      const double vr = r >= k0 ? v[r] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + u * kQrWaves;
        if (j < K) dot[u] = fma(vr, A[(size_t)j * M + r], dot[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) dot[u] = c * wave_all_sum(dot[u]);
    for (int r = (k0 & ~(kWave - 1)) + lane; r < M; r += kWave) {
      if (r < k0) continue;
      const double vr = v[r];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + u * kQrWaves;
        if (j < K) A[(size_t)j * M + r] = fma(-dot[u], vr, A[(size_t)j * M + r]);
      }
    }
  }
}

// As k_projection_regs for any M >= K, with the columns in global memory
// (A: qr_words(M, K)).  Q's columns replace the reflectors in place.
__global__ void __launch_bounds__(kQrThreads) k_projection(int M, int K,
                                                           const double* __restrict__ V,
                                                           double tiny, double* A,
                                                           double* __restrict__ P, int ldp,
                                                           int* __restrict__ bad,
                                                           int* __restrict__ bad_host) {
  __shared__ int stop;
  double* R = A + (size_t)K * M;
  double* vv = R + (size_t)K * K;
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  if (t == 0) stop = 0;
  for (int64_t e = t; e < (int64_t)M * K; e += kQrThreads)
    A[(e % K) * M + e / K] = V[e];
  __syncthreads();
  for (int k = 0; k < K; ++k) {
    double* v = A + (size_t)k * M;
    if (w == k % kQrWaves) {
      double s = 0.0;
      for (int r = lane; r < M; r += kWave)
        if (r >= k) s = fma(v[r], v[r], s);
      s = wave_all_sum(s);
      const double nrm = sqrt(s), vk = v[k];
      const double alpha = vk > 0 ? -nrm : nrm;
      if (lane == 0) {
        if (!(nrm > tiny)) stop = 1;
        R[(size_t)k * K + k] = alpha;
        v[k] = vk - alpha;
        vv[k] = 1.0 / (s + fabs(vk) * nrm);
      }
    }
    __syncthreads();
    if (stop) {
      if (t == 0) *bad = *bad_host = 1;
      return;
    }
    // the wave of column j is j mod 16: its first column past k
    reflect(M, K, k + 1 + (w + kQrWaves - (k + 1) % kQrWaves) % kQrWaves, k, vv[k], v, A);
  }
  __syncthreads();
  for (int64_t e = t; e < (int64_t)K * K; e += kQrThreads) {
    const int64_t i = e / K, j = e % K;
    if (i < j) R[e] = A[j * M + i];
  }
  for (int k = K - 1; k >= 0; --k) {
    __syncthreads();
    double* v = A + (size_t)k * M;
    reflect(M, K, k + 1 + (w + kQrWaves - (k + 1) % kQrWaves) % kQrWaves, k, vv[k], v, A);
    const double vk = v[k];
    __syncthreads();
    if (w == k % kQrWaves) {  // column k of Q: H_k e_k, in place of its reflector
      const double c = vv[k] * vk;
      for (int r = lane; r < M; r += kWave)
        v[r] = r < k ? 0.0 : (r == k ? 1.0 : 0.0) - c * v[r];
    }
  }
  __syncthreads();
  for (int m = t; m < M; m += kQrThreads)
    for (int i = K - 1; i >= 0; --i) {
      double s[4] = {A[(size_t)i * M + m], 0.0, 0.0, 0.0};
      int j = i + 1;
      for (; j + 4 <= K; j += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          s[u] = fma(-R[(size_t)i * K + j + u], A[(size_t)(j + u) * M + m], s[u]);
      for (; j < K; ++j) s[0] = fma(-R[(size_t)i * K + j], A[(size_t)j * M + m], s[0]);
      const double p = ((s[0] + s[1]) + (s[2] + s[3])) / R[(size_t)i * K + i];
      A[(size_t)i * M + m] = p;
      P[(size_t)i * ldp + m] = p;
    }
  if (t == 0) *bad = *bad_host = 0;
}

// C (R x n) = A (R x K) B (K x n), B and C row-major with leading dimension
// n, on the FP64 matrix cores.  A wave takes 16 columns and up to 64 rows
// (four 16 x 16 tiles), so B is read once per 64 rows; A's rows are staged
// through LDS 32 columns at a time, the next 32 and their values of B in
// flight meanwhile.  216 points, 56 terms and 32,768 outputs: 71 MB and 0.9
// GFLOP with the padding, 13 us at a copy's rate and 12 at the matrix cores';
// it takes 28, and 14 for 60 test points (80 together with one thread per
// column and 16 rows, which read B four times and A from LDS for every
// product).
// v_mfma_f64_16x16x4f64: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16];
// accumulator r of lane l is C[l / 16 + 4 r][l % 16].
typedef double double4_t __attribute__((ext_vector_type(4)));
constexpr int kRowTiles = 4, kWideRows = 16 * kRowTiles;  // most rows of a workgroup
constexpr int kWideCols = 16 * (kBlock / kWave);          // columns of a workgroup
constexpr int kWideK = 32;                                // staged depth

// A as this kernel reads it: rows of wide_ld(K) values, zero past K, and
// wide_rows(R) of them, whatever stands past R (such rows are not stored).
inline int wide_ld(int K) { return (K + kWideK - 1) / kWideK * kWideK; }
inline int wide_rows(int R) { return (R + kWideRows - 1) / kWideRows * kWideRows; }

// TILES: 16-row tiles of a workgroup (kRowTiles, or all of a smaller R's).
// skip (may be NULL): C is left alone if it holds nonzero.  The first workgroup's
// columns start at c0.
template <int TILES>
__global__ void __launch_bounds__(kBlock) k_small_times_wide(int R, int K, int lda, long long n,
                                                             long long c0,
                                                             const double* __restrict__ A,
                                                             const double* __restrict__ B,
                                                             double* __restrict__ C,
                                                             const int* __restrict__ skip) {
  // 36 doubles per row: the 64 lanes of an operand read fall on every bank twice
  constexpr int kPitch = kWideK + 4;
  constexpr int kA = 16 * TILES * kWideK / kBlock, kB = kWideK / 4;  // values per thread
  __shared__ double a[2][16 * TILES][kPitch];
  const int t = threadIdx.x, lane = t % kWave, i = lane % 16, kq = lane / 16;
  const long long c = c0 + (long long)blockIdx.x * kWideCols + (t / kWave) * 16 + i;
  const int r0 = blockIdx.y * kWideRows;
  if (skip && *skip) return;
  const double* b0 = B + (c < n ? c : n - 1);  // columns past n repeat the last one, unstored
  const int ar = t / kWideK, ak = t % kWideK;
  const double* a0 = A + (size_t)(r0 + ar) * lda + ak;
  double va[kA], vb[kB], b[kB];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const int k = k0 + 4 * u + kq;
      vb[u] = b0[(size_t)(k < K ? k : K - 1) * n];
    }
#pragma unroll
    for (int u = 0; u < kA; ++u) va[u] = a0[(size_t)u * (kBlock / kWideK) * lda + k0];
  };
  double4_t acc[TILES];
#pragma unroll
  for (int q = 0; q < TILES; ++q) acc[q] = double4_t{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int k0 = 0, p = 0; k0 < K; k0 += kWideK, p ^= 1) {
#pragma unroll
    for (int u = 0; u < kA; ++u) a[p][ar + u * (kBlock / kWideK)][ak] = va[u];
#pragma unroll
    for (int u = 0; u < kB; ++u) b[u] = k0 + 4 * u + kq < K ? vb[u] : 0.0;
    __syncthreads();  // the other buffer's readers passed the barrier before
    if (k0 + kWideK < K) fetch(k0 + kWideK);
#pragma unroll
    for (int u = 0; u < kB; ++u)
#pragma unroll
      for (int q = 0; q < TILES; ++q)
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p][16 * q + i][4 * u + kq], b[u], acc[q], 0,
                                                      0, 0);
  }
  if (c >= n) return;
#pragma unroll
  for (int q = 0; q < TILES; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = r0 + 16 * q + kq + 4 * r;
      if (row < R) C[(size_t)row * n + c] = acc[q][r];
    }
}

// Per output: mean W_0, variance sum_{i>0} W_i^2, and for each input j the
// first-order (terms in j alone) and total (terms involving j) shares.
// mask[i] bit j: term i involves input j; bit 30: it involves one input only.
// A workgroup takes 64 outputs; its four waves take every fourth term each
// (32,768 outputs alone would leave half the compute units without a
// workgroup), and every coefficient is read once for all inputs: 7 us
// at 56 terms and 3 inputs, 35 with a pass over the terms per input.  The first
// workgroup's outputs start at c0.
template <int D>
__global__ void __launch_bounds__(kBlock) k_pce_stats(int n_terms, int d, long long n,
                                                      long long c0,
                                                      const double* __restrict__ W,
                                                      const int* __restrict__ mask,
                                                      double* __restrict__ mean,
                                                      double* __restrict__ var,
                                                      double* __restrict__ first,
                                                      double* __restrict__ total) {
  constexpr int kParts = kBlock / kWave;
  __shared__ double part[kParts][kWave];
  const int lane = threadIdx.x % kWave;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const long long c = c0 + (long long)blockIdx.x * kWave + lane;
  const double* col = W + (c < n ? c : n - 1);
  double v = 0.0, f[D], t[D];
#pragma unroll
  for (int j = 0; j < D; ++j) f[j] = t[j] = 0.0;
  for (int i0 = 1 + w; i0 < n_terms; i0 += 4 * kParts) {
    double x[4];
    int m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * kParts;
      m[u] = i < n_terms ? mask[i] : 0;
      x[u] = i < n_terms ? col[(size_t)i * n] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double q = x[u] * x[u];
      v += q;
#pragma unroll
      for (int j = 0; j < D; ++j)
        if (m[u] & (1 << j)) {
          t[j] += q;
          if (m[u] & (1 << 30)) f[j] += q;
        }
    }
  }
  // the waves' sums, added in wave order; the first wave stores
  auto add = [&](double s) {
    __syncthreads();
    part[w][lane] = s;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int k = 0; k < kParts; ++k) r += part[k][lane];
    return r;
  };
  v = add(v);
  const bool store = w == 0 && c < n;
  if (store) {
    mean[c] = W[c];
    var[c] = v;
  }
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const double fj = add(f[j]), tj = add(t[j]);
    if (store && j < d) {
      first[(size_t)j * n + c] = v > 0 ? fj / v : 0.0;
      total[(size_t)j * n + c] = v > 0 ? tj / v : 0.0;
    }
  }
}

// Outputs of one launch: 64 of them take 256 threads, and a grid holds at most
// 2^32 along a dimension.
constexpr long long kOutPart = 1ll << 29;

// C (R x n) = A (R x K) B (K x n), A padded as k_small_times_wide reads it.
void small_times_wide(hipStream_t st, int R, int K, long long n, const double* A, const double* B,
                      double* C, const int* skip) {
  if (n == 0 || R == 0) return;
  require((n + kBlock - 1) / kBlock <= INT32_MAX, PPE_ERR_ARG, "too many outputs");
  auto run = [&](auto kernel) {
    for (long long c0 = 0; c0 < n; c0 += kOutPart) {
      const long long gx = (std::min(n - c0, kOutPart) + kWideCols - 1) / kWideCols;
      hipLaunchKernelGGL(kernel, dim3((unsigned)gx, (R + kWideRows - 1) / kWideRows), dim3(kBlock),
                         0, st, R, K, wide_ld(K), n, c0, A, B, C, skip);
      PPE_LAUNCH_CHECK();
    }
  };
  if (R <= 16)
    run(k_small_times_wide<1>);
  else if (R <= 32)
    run(k_small_times_wide<2>);
  else if (R <= 48)
    run(k_small_times_wide<3>);
  else
    run(k_small_times_wide<kRowTiles>);
}

// Queues P (K x M, rows of ldp) = R^-1 Q^T of V (M x K), both on the device;
// *bad as k_projection leaves it.
void projection(ppe_pce* q, int M, int K, const double* V, double tiny, double* P, int ldp,
                int* bad) {
  const size_t words = qr_words(M, K);
  if (!q->lds_max) {
    int v = 0;
    PPE_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, q->device));
    q->lds_max = (size_t)v;
  }
  if (M <= kWave * kQrRows && K <= kQrWaves * kQrCols &&
      words * sizeof(double) + 64 <= q->lds_max)
    hipLaunchKernelGGL(k_projection_regs, dim3(1), dim3(kQrThreads), words * sizeof(double),
                       q->stream, M, K, V, tiny, P, ldp, bad, q->bad_h);
  else
    hipLaunchKernelGGL(k_projection, dim3(1), dim3(kQrThreads), 0, q->stream, M, K, V, tiny,
                       q->qr_dev.get<double>(words), P, ldp, bad, q->bad_h);
  PPE_LAUNCH_CHECK();
}

__global__ void k_zero(int64_t n, double* __restrict__ p) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e < n) p[e] = 0.0;
}

// V [M x n_terms] in rows of ld values, `rows` of them (zero past M and past
// n_terms).
std::vector<double> vandermonde(const ppe_pce* q, int M, const double* xi, int ld, int rows) {
  const int K = q->n_terms, d = q->d, D = q->degree + 1;
  std::vector<double> V((size_t)rows * ld, 0.0), ps((size_t)d * D);
  for (int m = 0; m < M; ++m) {
    // psi_k of every input up to the degree
    for (int j = 0; j < d; ++j) {
      double pm = 0.0, p = 1.0;
      ps[(size_t)j * D] = 1.0;
      for (int k = 0; k < q->degree; ++k) {
        const double next = (xi[(size_t)m * d + j] * p - rec_b(q->kinds[j], k) * pm) /
                            rec_b(q->kinds[j], k + 1);
        pm = p;
        p = next;
        ps[(size_t)j * D + k + 1] = p;
      }
    }
    for (int i = 0; i < K; ++i) {
      double v = 1.0;
      for (int j = 0; j < d; ++j) v *= ps[(size_t)j * D + q->alpha[(size_t)i * d + j]];
      V[(size_t)m * ld + i] = v;
    }
  }
  return V;
}

}  // namespace
}  // namespace ppe

using ppe::require;

namespace {
template <class F>
ppe_status guarded_pce(ppe_pce* q, F&& f) {
  try {
    if (q) q->err.clear();
    return f();
  } catch (const ppe::Error& e) {
    if (q) q->err = e.what();
    return e.status;
  } catch (const std::bad_alloc&) {
    if (q) q->err = "host allocation failed";
    return PPE_ERR_OOM;
  } catch (const std::exception& e) {
    if (q) q->err = e.what();
    return PPE_ERR_INTERNAL;
  }
}
}  // namespace

extern "C" {

ppe_status ppe_pce_create(int32_t d, const int32_t* kinds, int32_t degree, void* stream,
                          ppe_pce** out) {
  if (!out || !kinds || d < 1 || d > 16 || degree < 0 || degree > 30) return PPE_ERR_ARG;
  for (int j = 0; j < d; ++j)
    if (kinds[j] != PPE_INPUT_NORMAL && kinds[j] != PPE_INPUT_UNIFORM) return PPE_ERR_ARG;
  auto* q = new ppe_pce();
  q->d = d;
  q->degree = degree;
  q->kinds.assign(kinds, kinds + d);
  q->stream = static_cast<hipStream_t>(stream);
  (void)hipGetDevice(&q->device);
  // graded order: by total degree, then lexicographically descending
  for (int deg = 0; deg <= degree; ++deg) {
    std::vector<std::vector<int>> lvl;
    std::vector<int> a(d, 0);
    std::function<void(int, int)> rec = [&](int j, int left) {
      if (j == d - 1) {
        a[j] = left;
        lvl.push_back(a);
        return;
      }
      for (int v = left; v >= 0; --v) {
        a[j] = v;
        rec(j + 1, left - v);
      }
    };
    rec(0, deg);
    for (auto& m : lvl) q->alpha.insert(q->alpha.end(), m.begin(), m.end());
  }
  q->n_terms = (int)(q->alpha.size() / d);
  *out = q;
  return PPE_OK;
}

void ppe_pce_destroy(ppe_pce* q) { delete q; }

int32_t ppe_pce_num_terms(const ppe_pce* q) { return q ? q->n_terms : 0; }

const char* ppe_pce_last_error(const ppe_pce* q) { return q ? q->err.c_str() : ""; }

ppe_status ppe_pce_terms(const ppe_pce* q, int32_t* alpha) {
  if (!q || !alpha) return PPE_ERR_ARG;
  std::copy(q->alpha.begin(), q->alpha.end(), alpha);
  return PPE_OK;
}

ppe_status ppe_pce_nodes(ppe_pce* q, int32_t grid, int32_t level, int32_t* n_nodes, double* nodes,
                         double* weights) {
  if (!q || !n_nodes) return PPE_ERR_ARG;
  return guarded_pce(q, [&]() -> ppe_status {
    require(level >= 1 && level <= 20, PPE_ERR_ARG, "level must be in 1..20");
    require(grid == PPE_GRID_TENSOR || grid == PPE_GRID_SMOLYAK, PPE_ERR_ARG, "unknown grid");
    const int d = q->d;
    ppe::NodeSet S;
    if (grid == PPE_GRID_TENSOR) {
      ppe::add_tensor(S, q->kinds, std::vector<int>(d, level), 1.0);
    } else {
      const int qq = level + d - 1;
      std::vector<int> idx(d, 1);
      for (;;) {
        int s = 0;
        for (int v : idx) s += v;
        if (s >= level && s <= qq) {
          const double c = ((qq - s) % 2 ? -1.0 : 1.0) * (double)ppe::binom(d - 1, qq - s);
          ppe::add_tensor(S, q->kinds, idx, c);
        }
        int j = 0;
        while (j < d && ++idx[j] > level) idx[j++] = 1;
        if (j == d) break;
      }
    }
    const int n = (int)S.pts.size();
    if (nodes) {
      require(*n_nodes >= n, PPE_ERR_ARG, "node arrays too small");
      int i = 0;
      for (auto& kv : S.pts) {
        for (int j = 0; j < d; ++j) nodes[(size_t)i * d + j] = kv.second.first[j];
        if (weights) weights[i] = kv.second.second;
        ++i;
      }
    }
    *n_nodes = n;
    return PPE_OK;
  });
}

ppe_status ppe_pce_fit(ppe_pce* q, int32_t M, const double* xi, int64_t n_out, const double* Y,
                       double* W) {
  if (!q) return PPE_ERR_ARG;
  return guarded_pce(q, [&]() -> ppe_status {
    require(xi && Y && W, PPE_ERR_ARG, "NULL array");
    require(M >= q->n_terms, PPE_ERR_ARG, "fewer sample points than expansion terms");
    require(n_out >= 0, PPE_ERR_ARG, "negative output count");
    const std::vector<double> V = ppe::vandermonde(q, M, xi, q->n_terms, M);
    double vmax = 0.0;
    for (double v : V) vmax = std::max(vmax, std::fabs(v));
    if (!q->bad_h) PPE_HIP(hipHostMalloc(reinterpret_cast<void**>(&q->bad_h), sizeof(int)));
    const int K = q->n_terms, ldp = ppe::wide_ld(M);
    const size_t len = V.size(), plen = (size_t)ppe::wide_rows(K) * ldp;
    if (ppe::host_projection(M, K)) {
      std::vector<double> P((size_t)K * ldp, 0.0);
      require(ppe::projection_host(M, K, V.data(), 1e-13 * vmax, P.data(), ldp), PPE_ERR_ARG,
              "the Vandermonde matrix of these points is rank deficient");
      double* Pd = q->a_dev.get<double>(plen);
      PPE_HIP(hipMemcpyAsync(Pd, P.data(), sizeof(double) * P.size(), hipMemcpyHostToDevice,
                             q->stream));
      ppe::small_times_wide(q->stream, K, M, n_out, Pd, Y, W, nullptr);
      PPE_HIP(hipStreamSynchronize(q->stream));
      return PPE_OK;
    }
    double* Pd = q->a_dev.get<double>(plen + len + 1);
    double* Vd = Pd + plen;
    int* bad = reinterpret_cast<int*>(Vd + len);
    PPE_HIP(hipMemcpyAsync(Vd, V.data(), sizeof(double) * len, hipMemcpyHostToDevice, q->stream));
    hipLaunchKernelGGL(ppe::k_zero, dim3(ppe::grid_for((int64_t)plen)), dim3(ppe::kBlock), 0,
                       q->stream, (int64_t)plen, Pd);
    PPE_LAUNCH_CHECK();
    ppe::projection(q, M, K, Vd, 1e-13 * vmax, Pd, ldp, bad);
    ppe::small_times_wide(q->stream, K, M, n_out, Pd, Y, W, bad);
    PPE_HIP(hipStreamSynchronize(q->stream));
    require(*q->bad_h == 0, PPE_ERR_ARG,
            "the Vandermonde matrix of these points is rank deficient");
    return PPE_OK;
  });
}

ppe_status ppe_pce_eval(ppe_pce* q, int32_t T, const double* xi, int64_t n_out, const double* W,
                        double* Y) {
  if (!q) return PPE_ERR_ARG;
  return guarded_pce(q, [&]() -> ppe_status {
    require(xi && W && Y, PPE_ERR_ARG, "NULL array");
    require(T >= 0 && n_out >= 0, PPE_ERR_ARG, "negative size");
    if (T == 0) return PPE_OK;
    const std::vector<double> V =
        ppe::vandermonde(q, T, xi, ppe::wide_ld(q->n_terms), ppe::wide_rows(T));
    double* Vd = q->a_dev.get<double>(V.size());
    PPE_HIP(hipMemcpyAsync(Vd, V.data(), sizeof(double) * V.size(), hipMemcpyHostToDevice, q->stream));
    ppe::small_times_wide(q->stream, T, q->n_terms, n_out, Vd, W, Y, nullptr);
    PPE_HIP(hipStreamSynchronize(q->stream));
    return PPE_OK;
  });
}

ppe_status ppe_pce_stats(ppe_pce* q, int64_t n_out, const double* W, double* mean, double* var,
                         double* first, double* total) {
  if (!q) return PPE_ERR_ARG;
  return guarded_pce(q, [&]() -> ppe_status {
    require(W && mean && var && first && total, PPE_ERR_ARG, "NULL array");
    require(n_out >= 0, PPE_ERR_ARG, "negative output count");
    if (n_out == 0) return PPE_OK;
    std::vector<int> mask(q->n_terms, 0);
    for (int i = 0; i < q->n_terms; ++i) {
      int cnt = 0;
      for (int j = 0; j < q->d; ++j)
        if (q->alpha[(size_t)i * q->d + j]) {
          mask[i] |= 1 << j;
          ++cnt;
        }
      if (cnt == 1) mask[i] |= 1 << 30;
    }
    int* md = q->mask_dev.get<int>(mask.size());
    PPE_HIP(hipMemcpyAsync(md, mask.data(), sizeof(int) * mask.size(), hipMemcpyHostToDevice, q->stream));
    require((n_out + ppe::kBlock - 1) / ppe::kBlock <= INT32_MAX, PPE_ERR_ARG, "too many outputs");
    auto run = [&](auto kernel) {
      for (long long c0 = 0; c0 < n_out; c0 += ppe::kOutPart) {
        const long long g =
            (std::min<long long>(n_out - c0, ppe::kOutPart) + ppe::kWave - 1) / ppe::kWave;
        hipLaunchKernelGGL(kernel, dim3((unsigned)g), dim3(ppe::kBlock), 0, q->stream, q->n_terms,
                           q->d, (long long)n_out, c0, W, md, mean, var, first, total);
        PPE_LAUNCH_CHECK();
      }
    };
    if (q->d <= 4)
      run(ppe::k_pce_stats<4>);
    else
      run(ppe::k_pce_stats<16>);
    PPE_HIP(hipStreamSynchronize(q->stream));
    return PPE_OK;
  });
}

}  // extern "C"
