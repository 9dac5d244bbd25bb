// Smoothed-aggregation AMG setup on the device (the multigrid of section 2.5
// of the paper, which coarsens the matrix by heuristics without a physical
// grid; the paper names no variant, this is smoothed aggregation):
//
//   strength   j strong for i  iff  a_ij^2 >= theta_l^2 (a_ii a_jj), j != i,
//              theta_l = theta theta_decay^l on level l (finest l = 0)
//   MIS-2      synchronous rounds over keys (state, fmix32(i ^ salt), -i):
//              an undecided node that holds the maximum key of its
//              distance-2 neighbourhood joins, one that sees a member there
//              leaves; nodes without strong neighbours never take part
//   aggregates member roots; strong neighbours of a root join it; leftovers
//              join the first-pass neighbour with the largest |a_ij|
//              (ties to the lowest index)
//   P_tent     B restricted to each aggregate, normalised; coarse B = norms
//   rho        Gershgorin bound on the finest level, 1.1 x a 15-step power
//              estimate of lambda_max(D^-1 A) on coarse levels
//   P          P_tent - (4 / (3 rho)) D^-1 A P_tent;  R = P^T;  A_c = R (A P)
//   coarsest   at most coarse_max rows: explicit inverse (Gauss-Jordan)
//
// Every product is formed row by row in a fixed order (Gustavson order: the
// entries of the left factor's row in ascending column order), so the setup
// is bitwise reproducible from run to run.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace ppe {
namespace {

constexpr int kPowerIters = 15;
constexpr double kPowerSafety = 1.1;
constexpr int kDenseMax = 1024;

// Deferred setup checks: bits of an error word read back with the spectral
// bounds once the hierarchy is built.  Kernels between a failed check and the
// read stay in bounds (an unassigned node only leaves its prolongator row
// empty; a lost diagonal or a non-positive pivot only spoils values).
enum SetupErr : int { SE_DIAG = 1, SE_DENSE = 2, SE_AGG = 4 };

enum : int { S_OUT = 0, S_UND = 1, S_IN = 2 };

// Row kernels below give each row a group of LPR lanes (LPR = power of two
// near the mean row length); lanes stride over the row's entries and the
// group combines its results with shuffles, in a fixed order.
template <int LPR, class T>
__device__ __forceinline__ T group_sum(T v) {
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_down(v, o, LPR);
  return v;
}

template <int LPR, class T>
__device__ __forceinline__ T group_max(T v) {
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) {
    T w = __shfl_down(v, o, LPR);
    v = w > v ? w : v;
  }
  return v;
}

// ------------------------------------------------------------------ strength
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_strength(int n, const int* __restrict__ rp,
                                                     const int* __restrict__ ci,
                                                     const double* __restrict__ v,
                                                     const double* __restrict__ diag, double theta2,
                                                     unsigned char* __restrict__ strong,
                                                     unsigned char* __restrict__ state) {
  const int i = (xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  int deg = 0;
  if (i < n) {
    const double di = diag[i];
    for (int k = rp[i] + lane; k < rp[i + 1]; k += LPR) {
      const int j = ci[k];
      const double a = v[k];
      const bool st = (j != i) && (a != 0.0) && (a * a >= theta2 * (di * diag[j]));
      strong[k] = st ? 1 : 0;
      deg += st ? 1 : 0;
    }
  }
  deg = group_sum<LPR>(deg);
  if (i < n && lane == 0) state[i] = deg > 0 ? S_UND : S_OUT;
}

// ------------------------------------------------------------------ MIS-2
__device__ __forceinline__ unsigned long long mis_key(unsigned char st, int j, uint32_t salt) {
  return ((unsigned long long)st << 62) |
         ((unsigned long long)fmix32((uint32_t)j ^ salt) << 30) |
         (unsigned long long)((1u << 30) - 1u - (uint32_t)j);
}

// m1_i = max key over i and its strong neighbours
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_mis_max1(int n, const int* __restrict__ rp,
                                                     const int* __restrict__ ci,
                                                     const unsigned char* __restrict__ strong,
                                                     const unsigned char* __restrict__ state,
                                                     uint32_t salt,
                                                     unsigned long long* __restrict__ m1) {
  const int i = (xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  unsigned long long m = 0;
  if (i < n) {
    for (int k = rp[i] + lane; k < rp[i + 1]; k += LPR) {
      if (!strong[k]) continue;
      const int j = ci[k];
      const unsigned long long kj = mis_key(state[j], j, salt);
      m = kj > m ? kj : m;
    }
  }
  m = group_max<LPR>(m);
  if (i < n && lane == 0) {
    const unsigned long long own = mis_key(state[i], i, salt);
    m1[i] = own > m ? own : m;
  }
}

// m2_i = max m1 over i and its strong neighbours; an undecided node joins if
// m2 is its own key, leaves if m2 belongs to a member.  *undecided is set to
// 1 if any node stays undecided.
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_mis_max2(int n, const int* __restrict__ rp,
                                                     const int* __restrict__ ci,
                                                     const unsigned char* __restrict__ strong,
                                                     unsigned char* __restrict__ state,
                                                     uint32_t salt,
                                                     const unsigned long long* __restrict__ m1,
                                                     int* __restrict__ undecided) {
  const int i = (xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  const bool und = i < n && state[i] == S_UND;
  unsigned long long m = 0;
  if (und) {
    for (int k = rp[i] + lane; k < rp[i + 1]; k += LPR) {
      if (!strong[k]) continue;
      const unsigned long long mj = m1[ci[k]];
      m = mj > m ? mj : m;
    }
  }
  m = group_max<LPR>(m);
  int left = 0;
  if (und && lane == 0) {
    const unsigned long long mm = m1[i] > m ? m1[i] : m;
    if (mm == mis_key(S_UND, i, salt))
      state[i] = S_IN;
    else if ((mm >> 62) == S_IN)
      state[i] = S_OUT;
    else
      left = 1;
  }
  // the host only asks whether any node is still undecided: a plain store of
  // the same value from every such block (same-address atomics from every
  // block serialise across the chip)
  left = block_sum<kBlock>(left);
  if (threadIdx.x == 0 && left) *undecided = 1;
}

// ------------------------------------------------------------------ finest level, ELL
// The same strength, MIS-2 and joining rules on the finest level's
// slot-major ELL copy of the off-diagonal part (slot k of row i at
// k n + i, padding = the row itself): one thread per row, every slot's load
// issued before its gathers, no row pointers.  The strength pass leaves
// scol = the column of each strong entry and the row itself elsewhere, so
// the later passes read one array.  Results are maxima and per-entry tests,
// as in the CSR kernels, so they are the same bit for bit.
template <int WM>
__device__ __forceinline__ void slot_cols(int i, int n, int W, const int* __restrict__ col,
                                          int (&c)[WM]) {
#pragma unroll
  for (int k = 0; k < WM; ++k) c[k] = k < W ? col[(size_t)k * n + i] : i;
}

// WM: unrolled slot count covering W (0: a plain loop over W slots).
template <int WM>
__global__ void __launch_bounds__(kBlock) k_strength_ell(int n, int W, const int* __restrict__ ecol,
                                                         const double* __restrict__ ev,
                                                         const double* __restrict__ diag,
                                                         double theta2, int* __restrict__ scol,
                                                         unsigned char* __restrict__ state) {
  const int i = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  const double di = diag[i];
  int deg = 0;
  auto test = [&](int k, int j) {
    const double a = ev[(size_t)k * n + i];
    const bool st = (j != i) && (a != 0.0) && (a * a >= theta2 * (di * diag[j]));
    scol[(size_t)k * n + i] = st ? j : i;
    deg += st ? 1 : 0;
  };
  if constexpr (WM > 0) {
    int c[WM];
    slot_cols<WM>(i, n, W, ecol, c);
#pragma unroll
    for (int k = 0; k < WM; ++k)
      if (k < W) test(k, c[k]);
  } else {
    for (int k = 0; k < W; ++k) test(k, ecol[(size_t)k * n + i]);
  }
  state[i] = deg > 0 ? S_UND : S_OUT;
}

template <int WM>
__global__ void __launch_bounds__(kBlock) k_mis_max1_ell(int n, int W, const int* __restrict__ scol,
                                                         const unsigned char* __restrict__ state,
                                                         uint32_t salt,
                                                         unsigned long long* __restrict__ m1) {
  const int i = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  unsigned long long m = mis_key(state[i], i, salt);
  auto take = [&](int j) {
    if (j == i) return;
    const unsigned long long kj = mis_key(state[j], j, salt);
    m = kj > m ? kj : m;
  };
  if constexpr (WM > 0) {
    int c[WM];
    slot_cols<WM>(i, n, W, scol, c);
#pragma unroll
    for (int k = 0; k < WM; ++k) take(c[k]);
  } else {
    for (int k = 0; k < W; ++k) take(scol[(size_t)k * n + i]);
  }
  m1[i] = m;
}

template <int WM>
__global__ void __launch_bounds__(kBlock) k_mis_max2_ell(int n, int W, const int* __restrict__ scol,
                                                         unsigned char* __restrict__ state,
                                                         uint32_t salt,
                                                         const unsigned long long* __restrict__ m1) {
  const int i = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n || state[i] != S_UND) return;
  unsigned long long m = m1[i];
  auto take = [&](int j) {
    if (j == i) return;
    const unsigned long long mj = m1[j];
    m = mj > m ? mj : m;
  };
  if constexpr (WM > 0) {
    int c[WM];
    slot_cols<WM>(i, n, W, scol, c);
#pragma unroll
    for (int k = 0; k < WM; ++k) take(c[k]);
  } else {
    for (int k = 0; k < W; ++k) take(scol[(size_t)k * n + i]);
  }
  if (m == mis_key(S_UND, i, salt))
    state[i] = S_IN;
  else if ((m >> 62) == S_IN)
    state[i] = S_OUT;
}

// ------------------------------------------------------------------ MIS-2, last rounds
// The set is the greedy one in descending key order whatever the schedule: a
// node is in if no node of a higher key within distance 2 is in.  So once few
// nodes are undecided they need no synchronous rounds over all rows: each
// looks at its distance-2 neighbourhood itself and decides in place, leaving
// when a member is there, joining when every node of a higher key there has
// left, and waiting for the next dispatch otherwise.  States only go from
// undecided to decided, so an old one read here makes a node wait, never
// decide wrongly.  *undecided is set to 1 if any node waits.  A block gathers
// the undecided nodes of its rows in LDS and gives each eight lanes: with a lane
// per node most lanes idle over chains of dependent loads.  A round over the
// 1.47 M rows of a 128^3 system takes 25 us and the set 15 of them; now six, and
// nine of these of 12 down to 5 us.  Coarse levels keep their rounds: a node
// there has hundreds of neighbours within distance 2, and a dispatch took 18 to
// 96 us where a round takes 8 to 22.
constexpr int kMisRounds = 6;  // rounds over all rows first: 1 to 2% are left
constexpr int kFinishRows = 2048;  // rows per block

__device__ __forceinline__ unsigned char state_of(const unsigned char* state, int j) {
  return __hip_atomic_load(state + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void decide(unsigned char* state, int i, unsigned char st) {
  __hip_atomic_store(state + i, st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// what node j means to an undecided node of key own: bit 0 a member, bit 1 wait
__device__ __forceinline__ int mis_look(const unsigned char* state, int j, uint32_t salt,
                                        unsigned long long own) {
  const unsigned char st = state_of(state, j);
  return st == S_IN ? 1 : (st == S_UND && mis_key(S_UND, j, salt) > own ? 2 : 0);
}

template <int WM>
__global__ void __launch_bounds__(kBlock) k_mis_finish_ell(int n, int W,
                                                           const int* __restrict__ scol,
                                                           unsigned char* state, uint32_t salt,
                                                           int* __restrict__ undecided) {
  __shared__ int list[kFinishRows], num;
  if (threadIdx.x == 0) num = 0;
  __syncthreads();
  const int first = xcd_block(blockIdx.x, gridDim.x) * kFinishRows + threadIdx.x;
#pragma unroll
  for (int u = 0; u < kFinishRows / kBlock; ++u) {
    const int i = first + u * kBlock;
    if (i < n && state_of(state, i) == S_UND) list[atomicAdd(&num, 1)] = i;
  }
  __syncthreads();
  const int l = threadIdx.x % 8;
  bool waits = false;
  for (int e = threadIdx.x / 8; e < num; e += kBlock / 8) {
    const int i = list[e];
    const unsigned long long own = mis_key(S_UND, i, salt);
    int seen = 0;
    for (int k = l; k < W; k += 8) {
      const int j = scol[(size_t)k * n + i];
      if (j == i) continue;
      if constexpr (WM > 0) {
        int d[WM];
        slot_cols<WM>(j, n, W, scol, d);  // padding holds j
#pragma unroll
        for (int q = 0; q < WM; ++q) seen |= mis_look(state, d[q], salt, own);
      } else {
        for (int q = 0; q < W; ++q) seen |= mis_look(state, scol[(size_t)q * n + j], salt, own);
      }
      seen |= mis_look(state, j, salt, own);
    }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) seen |= __shfl_xor(seen, o, 8);
    if (seen == 2) waits = true;
    else if (l == 0) decide(state, i, seen & 1 ? S_OUT : S_IN);
  }
  if (waits) *undecided = 1;
}

template <int WM>
__global__ void __launch_bounds__(kBlock) k_agg_first_ell(int n, int W, const int* __restrict__ scol,
                                                          const unsigned char* __restrict__ state,
                                                          const int* __restrict__ root_id,
                                                          int* __restrict__ agg1) {
  const int i = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  if (state[i] == S_IN) {
    agg1[i] = root_id[i];
    return;
  }
  int a = -1;
  auto take = [&](int j) {
    if (j != i && state[j] == S_IN) a = max(a, root_id[j]);
  };
  if constexpr (WM > 0) {
    int c[WM];
    slot_cols<WM>(i, n, W, scol, c);
#pragma unroll
    for (int k = 0; k < WM; ++k) take(c[k]);
  } else {
    for (int k = 0; k < W; ++k) take(scol[(size_t)k * n + i]);
  }
  agg1[i] = a;
}

template <int WM>
__global__ void __launch_bounds__(kBlock) k_agg_second_ell(int n, int W, const int* __restrict__ scol,
                                                           const double* __restrict__ ev,
                                                           const int* __restrict__ agg1,
                                                           int* __restrict__ agg,
                                                           int* __restrict__ flag) {
  const int i = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  int a = agg1[i];
  if (a < 0) {
    double best = -1.0;
    int bestj = INT32_MAX, any = 0;
    auto take = [&](int k, int j) {
      if (j == i) return;
      any = 1;
      if (agg1[j] < 0) return;
      const double w = fabs(ev[(size_t)k * n + i]);
      if (w > best || (w == best && j < bestj)) { best = w; bestj = j; }
    };
    if constexpr (WM > 0) {
      int c[WM];
      slot_cols<WM>(i, n, W, scol, c);
#pragma unroll
      for (int k = 0; k < WM; ++k) take(k, c[k]);
    } else {
      for (int k = 0; k < W; ++k) take(k, scol[(size_t)k * n + i]);
    }
    if (best >= 0.0) a = agg1[bestj];
    else if (any) atomicOr(flag, SE_AGG);
  }
  agg[i] = a;
}

// Finest level: the smoothed prolongator P = P_tent - omega D^-1 Q, Q = A
// P_tent, from the ELL copy, one thread per row (omega as in k_smooth_p; a pass
// of its own took 54 us for 1.47 M rows, reading Q back).  P_tent
// has one entry per aggregated node (pt_j in column agg_j), so row i of Q
// holds, for every aggregate J reached from row i, the sum of a_ij pt_j
// over that row's entries j in J.  The row's entries are taken in CSR order
// (ascending column, the diagonal in its place) and each sum starts from 0
// in that order, as the general product's do (rows of P_tent have one entry):
// bitwise its result.  COUNT: distinct aggregates per row into counts; else the row, sorted by
// aggregate, at rp[i].
template <int WM, bool COUNT>
__global__ void __launch_bounds__(kBlock) k_coarsen_cols_ell(
    int n, int W, const int* __restrict__ ecol, const double* __restrict__ ev,
    const double* __restrict__ diag, const int* __restrict__ agg, const double* __restrict__ pt,
    const double* __restrict__ rho, int* __restrict__ counts, const int* __restrict__ rp,
    int* __restrict__ ci, double* __restrict__ v) {
  const int i = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  // fixed register slots: ELL slot k (aggregate Jk[k], -1 for none), and the
  // diagonal, which comes before slot dpos in CSR order
  int c[WM];
  slot_cols<WM>(i, n, W, ecol, c);
  int Jk[WM];
  double yk[WM];
  int dpos = WM;
#pragma unroll
  for (int k = WM - 1; k >= 0; --k) {
    const int j = c[k];
    const bool real = j != i;  // padding (slots past W included) holds the row
    if (real && j > i) dpos = k;
    Jk[k] = real ? agg[j] : -1;
    if (!COUNT) yk[k] = Jk[k] >= 0 ? ev[(size_t)k * n + i] * pt[j] : 0.0;
  }
  const int Jd = agg[i];
  const double di = COUNT ? 1.0 : diag[i], pti = !COUNT && Jd >= 0 ? pt[i] : 0.0;
  const double yd = Jd >= 0 ? di * pti : 0.0;
  const double omega = COUNT ? 0.0 : 4.0 / (3.0 * *rho), dinv = 1.0 / di;
  int out = COUNT ? 0 : rp[i];
  int last = -1;
  for (int step = 0; step <= WM; ++step) {
    int cur = Jd > last ? Jd : INT32_MAX;
#pragma unroll
    for (int k = 0; k < WM; ++k)
      if (Jk[k] > last && Jk[k] < cur) cur = Jk[k];
    if (cur == INT32_MAX) break;
    if (!COUNT) {
      double sum = 0.0;
#pragma unroll
      for (int k = 0; k <= WM; ++k) {
        if (k == dpos && Jd == cur) sum = sum + yd;
        if (k < WM && Jk[k] == cur) sum = sum + yk[k];
      }
      ci[out] = cur;
      v[out] = (cur == Jd ? pti : 0.0) - omega * (sum * dinv);
    }
    ++out;
    last = cur;
  }
  if (COUNT) counts[i] = out;
}

// Finest level: AP = A P by rows, one thread per row from the ELL copy:
// row i of AP merges the sorted rows of P selected by row i of A (its ELL
// slots and the diagonal, at most WM + 1 of them), column by column.  A
// column's products are added from 0 in CSR order of A's row (the general product
// may take the later entries of P's longer rows in a later turn, so the two agree
// to rounding).  COUNT: entries per row into counts; else the row, sorted, at
// rp[i].
// The next entries of each list wait in registers, loaded kApU at a time: the
// pass is bound by the accesses of 64 lanes to as many lines (one a cycle and
// compute unit), and a row of P is three to four entries.  P's arrays
// therefore extend kApU entries past its last.  Loaded one by one, each when the
// one before it was taken, 1.47 M rows took 411 us and take 231 (0.15 M rows: 27
// us either way).
constexpr int kApU = 4;
template <int U> struct __attribute__((packed, aligned(4))) ApCols { int c[U]; };
template <int U> struct __attribute__((packed, aligned(8))) ApVals { double v[U]; };
struct __attribute__((packed, aligned(4))) ApEnds { int first, end; };

template <int WM, bool COUNT>
__global__ void __launch_bounds__(kBlock) k_ap_merge_ell(
    int n, int W, const int* __restrict__ ecol, const double* __restrict__ ev,
    const double* __restrict__ diag, const int* __restrict__ prp, const int* __restrict__ pci,
    const double* __restrict__ pv, int* __restrict__ counts, const int* __restrict__ rp,
    int* __restrict__ ci, double* __restrict__ v) {
  constexpr int U = COUNT ? 1 : kApU;  // the count reads columns only
  const int i = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  int c[WM];
  slot_cols<WM>(i, n, W, ecol, c);
  // list k < WM: row c[k] of P (empty for padding); list WM: row i (the
  // diagonal), which comes before list dpos in CSR order
  int pos[WM + 1], end[WM + 1];
  ApCols<U> col[WM + 1];
  ApVals<U> val[WM + 1];
  double a[WM + 1];
  int dpos = WM;
#pragma unroll
  for (int k = WM; k >= 0; --k) {
    const int j = k < WM ? c[k] : i;
    const bool real = k == WM || j != i;
    if (k < WM && real && j > i) dpos = k;
    const ApEnds e = *reinterpret_cast<const ApEnds*>(prp + j);
    pos[k] = real ? e.first : 0;
    end[k] = real ? e.end : 0;
    if (!COUNT) a[k] = k < WM ? (real ? ev[(size_t)k * n + i] : 0.0) : diag[i];
  }
  auto load = [&](int k) {  // entries pos .. pos + U of list k, past its end none
    col[k] = *reinterpret_cast<const ApCols<U>*>(pci + pos[k]);
    if (!COUNT) val[k] = *reinterpret_cast<const ApVals<U>*>(pv + pos[k]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (pos[k] + u >= end[k]) col[k].c[u] = INT32_MAX;
    pos[k] += U;
  };
#pragma unroll
  for (int k = 0; k <= WM; ++k) load(k);
  int out = COUNT ? 0 : rp[i];
  for (;;) {
    int cur = col[0].c[0];
#pragma unroll
    for (int k = 1; k <= WM; ++k) cur = min(cur, col[k].c[0]);
    if (cur == INT32_MAX) break;
    if (!COUNT) {
      double sum = 0.0;
#pragma unroll
      for (int k = 0; k <= WM; ++k) {
        if (k == dpos && col[WM].c[0] == cur) sum = sum + a[WM] * val[WM].v[0];
        if (k < WM && col[k].c[0] == cur) sum = sum + a[k] * val[k].v[0];
      }
      ci[out] = cur;
      v[out] = sum;
    }
    ++out;
#pragma unroll
    for (int k = 0; k <= WM; ++k)
      if (col[k].c[0] == cur) {
#pragma unroll
        for (int u = 0; u + 1 < U; ++u) {
          col[k].c[u] = col[k].c[u + 1];
          if (!COUNT) val[k].v[u] = val[k].v[u + 1];
        }
        col[k].c[U - 1] = INT32_MAX;
        if (col[k].c[0] == INT32_MAX && pos[k] < end[k]) load(k);
      }
  }
  if (COUNT) counts[i] = out;
}

// ------------------------------------------------------------------ MIS-2, small levels
// All rounds of a level whose strong graph fits in one workgroup's LDS, and
// the numbering of its roots: the same synchronous rounds as above on keys
// (state included) held in LDS, columns in 16 bits.  A round's two passes are
// 3 to 4 us each as dispatches whatever the level's size, and the host reads
// the undecided count after a guessed number of them; here a round is two
// barriers and one compute unit's LDS reads, 0.1 us per 400 entries and pass.
// So it pays up to about kMisEntries: 16^3 (2,816 rows of six slots, 13
// rounds) took 58 us in place of 30 dispatches and two or three round trips
// (assembly 702 -> 639 us), and takes 43 with the last nine rounds on the few
// undecided nodes, while a level of 605 rows and 47 k entries took
// 165 us here and takes 65 in dispatches.  LPR lanes per row; rows as slots
// (rp NULL: W columns of slot k at k n, the row itself = none) or CSR with the
// strong flags.
constexpr int64_t kMisEntries = 20480;
constexpr int kMisThreads = 1024;
constexpr int kMisSmallRounds = 4;  // rounds over all rows before the few left go alone
// What the kernel takes of a workgroup's LDS beside mis_small_lds: the
// wavefronts' sums and what the voting barriers use (328 bytes as built).
constexpr size_t kMisStatic = 1024;
inline size_t mis_small_lds(int64_t n, int64_t entries, bool csr) {
  return (size_t)(16 * n + (csr ? 4 * (n + 1) : 0) + 2 * entries);
}

__global__ void __launch_bounds__(kMisThreads) k_mis_small(
    int n, int lpr, int W, const int* __restrict__ scol, const int* __restrict__ rp,
    const int* __restrict__ ci, const unsigned char* __restrict__ strong, uint32_t salt,
    unsigned char* __restrict__ state, int* __restrict__ root_id, long long* __restrict__ n_roots) {
  extern __shared__ unsigned long long mis_lds[];
  __shared__ int wsum[kMisThreads / kWave];
  unsigned long long* key = mis_lds;
  unsigned long long* m1 = key + n;
  int* ptr = reinterpret_cast<int*>(m1 + n);  // CSR only
  unsigned short* col = reinterpret_cast<unsigned short*>(ptr + (rp ? n + 1 : 0));
  const int t = threadIdx.x, lane = t % lpr, groups = kMisThreads / lpr;
  for (int i = t; i < n; i += kMisThreads) key[i] = mis_key(state[i], i, salt);
  if (rp) {
    for (int i = t; i <= n; i += kMisThreads) ptr[i] = rp[i];
    __syncthreads();
    // a weak entry stores its row, whose key every maximum holds anyway
    for (int i = t / lpr; i < n; i += groups)
      for (int k = ptr[i] + lane; k < ptr[i + 1]; k += lpr)
        col[k] = (unsigned short)(strong[k] ? ci[k] : i);
  } else {
    for (int e = t; e < W * n; e += kMisThreads) col[e] = (unsigned short)scol[e];
  }
  __syncthreads();
  // the largest of v over row i and its strong neighbours, in every lane
  auto row_max = [&](int i, const unsigned long long* v) {
    unsigned long long m = v[i];
    int k = rp ? ptr[i] + lane : lane * n + i;
    const int k1 = rp ? ptr[i + 1] : W * n, step = rp ? lpr : lpr * n;
    for (; k + 3 * step < k1; k += 4 * step) {
      unsigned long long x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = v[col[k + u * step]];
#pragma unroll
      for (int u = 0; u < 4; ++u) m = x[u] > m ? x[u] : m;
    }
    for (; k < k1; k += step) {
      const unsigned long long x = v[col[k]];
      m = x > m ? x : m;
    }
    for (int o = lpr / 2; o > 0; o >>= 1) {
      const unsigned long long x = __shfl_xor(m, o, kWave);
      m = x > m ? x : m;
    }
    return m;
  };
  // every lane group runs the same trips, so that the shuffles see all lanes
  const int trips = (n + groups - 1) / groups;
  const bool slots = !rp && lpr == 1;
  bool finish = false;
  for (int round = 0;; ++round) {
    if (slots && round == kMisSmallRounds) {
      finish = true;
      break;
    }
    for (int q = 0; q < trips; ++q) {
      const int i = q * groups + t / lpr;
      const unsigned long long m = row_max(i < n ? i : n - 1, key);
      if (i < n && lane == 0) m1[i] = m;
    }
    __syncthreads();
    int und = 0;
    for (int q = 0; q < trips; ++q) {
      const int i = q * groups + t / lpr;
      const unsigned long long m = row_max(i < n ? i : n - 1, m1);
      if (i >= n || lane != 0) continue;
      const unsigned long long own = key[i];
      if ((own >> 62) != S_UND) continue;
      const unsigned long long low = own & ((1ull << 62) - 1ull);
      if (m == own)
        key[i] = ((unsigned long long)S_IN << 62) | low;
      else if ((m >> 62) == S_IN)
        key[i] = low;  // S_OUT
      else
        und = 1;
    }
    if (!__syncthreads_or(und)) break;
  }
  if (finish) {
    // the nodes left, eight lanes each, in place (as k_mis_finish_ell: a key is
    // read by one relaxed access, old or new); the one of the highest key among
    // them decides in every pass
    __shared__ int num;
    unsigned short* list = reinterpret_cast<unsigned short*>(m1);
    auto key_of = [&](int j) {
      return __hip_atomic_load(key + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto decide_key = [&](int i, unsigned long long k) {
      __hip_atomic_store(key + i, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    if (t == 0) num = 0;
    __syncthreads();
    for (int i = t; i < n; i += kMisThreads)
      if ((key[i] >> 62) == S_UND) list[atomicAdd(&num, 1)] = (unsigned short)i;
    __syncthreads();
    for (;;) {
      int und = 0;
      for (int e0 = 0; e0 < num; e0 += kMisThreads / 8) {
        const int e = e0 + t / 8, l = t % 8, i = e < num ? list[e] : 0;
        const unsigned long long own = key_of(i);
        const bool on = e < num && (own >> 62) == S_UND;
        unsigned long long m = own;
        if (on)
          for (int k = l; k < W; k += 8) {
            const int j = col[k * n + i];
            const unsigned long long kj = key_of(j);
            m = kj > m ? kj : m;
            for (int q = 0; q < W; ++q) {
              const unsigned long long x = key_of(col[q * n + j]);
              m = x > m ? x : m;
            }
          }
        for (int o = 4; o > 0; o >>= 1) {
          const unsigned long long x = __shfl_xor(m, o, kWave);
          m = x > m ? x : m;
        }
        if (!on || l != 0) continue;
        const unsigned long long low = own & ((1ull << 62) - 1ull);
        if (m == own)
          decide_key(i, ((unsigned long long)S_IN << 62) | low);
        else if ((m >> 62) == S_IN)
          decide_key(i, low);  // S_OUT
        else
          und = 1;
      }
      if (!__syncthreads_or(und)) break;
    }
  }
  // states out; roots numbered in row order (each thread a run of rows)
  const int per = (n + kMisThreads - 1) / kMisThreads, i0 = t * per, i1 = min(n, i0 + per);
  int cnt = 0;
  for (int i = i0; i < i1; ++i) {
    const int st = (int)(key[i] >> 62);
    state[i] = (unsigned char)st;
    cnt += st == S_IN ? 1 : 0;
  }
  int inc = cnt;
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(inc, o, kWave);
    if (t % kWave >= o) inc += u;
  }
  if (t % kWave == kWave - 1) wsum[t / kWave] = inc;
  __syncthreads();
  int at = inc - cnt, total = 0;
  for (int q = 0; q < kMisThreads / kWave; ++q) {
    if (q < t / kWave) at += wsum[q];
    total += wsum[q];
  }
  for (int i = i0; i < i1; ++i) {
    root_id[i] = at;
    at += (key[i] >> 62) == S_IN ? 1 : 0;
  }
  if (t == 0) {
    root_id[n] = total;
    *n_roots = total;
  }
}

// ------------------------------------------------------------------ aggregation
__global__ void k_is_root(int n, const unsigned char* __restrict__ state, int* __restrict__ root) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) root[i] = state[i] == S_IN ? 1 : 0;
}

// A root's id; a node with a strong root neighbour takes that root's id (the
// root is unique: roots are at least three edges apart); others -1.
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_agg_first(int n, const int* __restrict__ rp,
                                                      const int* __restrict__ ci,
                                                      const unsigned char* __restrict__ strong,
                                                      const unsigned char* __restrict__ state,
                                                      const int* __restrict__ root_id,
                                                      int* __restrict__ agg1) {
  const int i = (xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  int a = -1;
  const bool root = i < n && state[i] == S_IN;
  if (i < n && !root) {
    for (int k = rp[i] + lane; k < rp[i + 1]; k += LPR) {
      const int j = ci[k];
      if (strong[k] && state[j] == S_IN) a = root_id[j];
    }
  }
  a = group_max<LPR>(a);
  if (i < n && lane == 0) agg1[i] = root ? root_id[i] : a;
}

// Leftover nodes join the first-pass neighbour with the largest |a_ij|, ties
// to the lowest j.
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_agg_second(int n, const int* __restrict__ rp,
                                                       const int* __restrict__ ci,
                                                       const double* __restrict__ v,
                                                       const unsigned char* __restrict__ strong,
                                                       const int* __restrict__ agg1,
                                                       int* __restrict__ agg, int* __restrict__ flag) {
  const int i = (xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  const int a1 = i < n ? agg1[i] : 0;
  double best = -1.0;
  int bestj = INT32_MAX;
  int any = 0;
  if (i < n && a1 < 0) {
    for (int k = rp[i] + lane; k < rp[i + 1]; k += LPR) {
      if (!strong[k]) continue;
      any = 1;
      const int j = ci[k];
      if (agg1[j] < 0) continue;
      const double w = fabs(v[k]);
      if (w > best || (w == best && j < bestj)) { best = w; bestj = j; }
    }
  }
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) {
    const double wb = __shfl_down(best, o, LPR);
    const int jb = __shfl_down(bestj, o, LPR);
    if (wb > best || (wb == best && jb < bestj)) { best = wb; bestj = jb; }
  }
  any = group_max<LPR>(any);
  if (i < n && lane == 0) {
    int a = a1;
    if (a < 0) {
      if (best >= 0.0) a = agg1[bestj];
      else if (any) atomicOr(flag, SE_AGG);
    }
    agg[i] = a;
  }
}

__global__ void k_agg_fill(int n, const int* __restrict__ agg, const int* __restrict__ ptr,
                           const int* __restrict__ pos, int* __restrict__ mem) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n && agg[i] >= 0) mem[ptr[agg[i]] + pos[i]] = i;
}

// Sort each aggregate's members, then norm_J = sqrt(sum B_i^2) in ascending
// i.  One wavefront per aggregate.  Up to 64 members are ranked in
// registers; up to kAggLds by the whole wave (the members staged in LDS,
// each lane counts for its own members the smaller keys among all of them,
// then writes them back in rank order); a larger aggregate is sorted by
// one lane in place.  The squares are summed
// in rank order by one lane.
constexpr int kAggLds = 1024;
__global__ void __launch_bounds__(kBlock) k_agg_norm(int na, const int* __restrict__ ptr,
                                                     int* __restrict__ mem,
                                                     const double* __restrict__ B,
                                                     double* __restrict__ Bc) {
  __shared__ double sq[kBlock];
  __shared__ int skey[kBlock / kWave][kAggLds];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int J0 = 2 * (blockIdx.x * (kBlock / kWave) + w);
  if (J0 >= na) return;  // whole wavefronts: only wave-level ordering below
  double* wsq = sq + w * kWave;
  int* wk = skey[w];
  // a wavefront's LDS operations complete in issue order; the fences keep
  // the compiler from moving them across
  auto wave_sync = []() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // two aggregates of up to half a wavefront's lanes side by side: they have
  // some eleven members, and what a wavefront waits for is the chain from the
  // pointers to the squares (133 k aggregates 58 -> 34 us)
  constexpr int kHalf = kWave / 2;
  const int half = lane / kHalf, hl = lane % kHalf, Jh = J0 + half;
  const int bh = Jh < na ? ptr[Jh] : 0, mh = Jh < na ? ptr[Jh + 1] - bh : 0;
  if (__all(mh <= kHalf)) {
    const int key = hl < mh ? mem[bh + hl] : INT32_MAX;
    int rank = 0;
    for (int q = 0; __any(q < mh); ++q) rank += __shfl(key, q, kHalf) < key ? 1 : 0;
    if (hl < mh) {
      mem[bh + rank] = key;
      wsq[half * kHalf + rank] = B[key] * B[key];
    }
    wave_sync();
    if (hl == 0 && Jh < na) {
      double s = 0.0;
      for (int q = 0; q < mh; ++q) s = s + wsq[half * kHalf + q];
      Bc[Jh] = sqrt(s);
    }
    return;
  }
  for (int J = J0; J < min(J0 + 2, na); ++J) {
    const int b = ptr[J], e = ptr[J + 1], m = e - b;
    double s = 0.0;
    if (m <= kWave) {
      const int key = lane < m ? mem[b + lane] : INT32_MAX;
      int rank = 0;
      for (int q = 0; q < m; ++q) rank += __shfl(key, q, kWave) < key ? 1 : 0;
      if (lane < m) {
        mem[b + rank] = key;
        wsq[rank] = B[key] * B[key];
      }
      wave_sync();
      if (lane == 0)
        for (int q = 0; q < m; ++q) s = s + wsq[q];
    } else if (m <= kAggLds) {
      constexpr int T = kAggLds / kWave;  // members per lane
      int myk[T], myr[T];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int i = lane + t * kWave;
        myk[t] = i < m ? mem[b + i] : INT32_MAX;
        if (i < m) wk[i] = myk[t];
      }
      wave_sync();
#pragma unroll
      for (int t = 0; t < T; ++t) {
        int r = 0;
        if (lane + t * kWave < m)
          for (int q = 0; q < m; ++q) r += wk[q] < myk[t] ? 1 : 0;
        myr[t] = r;
      }
      wave_sync();  // every lane has read wk before it is overwritten in rank order
#pragma unroll
      for (int t = 0; t < T; ++t)
        if (lane + t * kWave < m) wk[myr[t]] = myk[t];
      wave_sync();
      for (int c = 0; c < m; c += kWave) {
        const int q = c + lane;
        if (q < m) {
          const int key = wk[q];
          mem[b + q] = key;
          wsq[lane] = B[key] * B[key];
        }
        wave_sync();
        if (lane == 0)
          for (int t = 0; t < kWave && c + t < m; ++t) s = s + wsq[t];
        wave_sync();  // wsq is rewritten for the next chunk
      }
    } else if (lane == 0) {
      for (int i = b + 1; i < e; ++i) {
        int key = mem[i], j = i - 1;
        while (j >= b && mem[j] > key) { mem[j + 1] = mem[j]; --j; }
        mem[j + 1] = key;
      }
      for (int i = b; i < e; ++i) s = s + B[mem[i]] * B[mem[i]];
    }
    if (lane == 0) Bc[J] = sqrt(s);
    wave_sync();  // LDS is rewritten for the next one
  }
}

__global__ void k_tent(int n, const int* __restrict__ agg, const double* __restrict__ B,
                       const double* __restrict__ Bc, int* __restrict__ cnt,
                       double* __restrict__ pt) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  int a = agg[i];
  cnt[i] = a >= 0 ? 1 : 0;
  pt[i] = a >= 0 ? B[i] / Bc[a] : 0.0;
}

__global__ void k_tent_csr(int n, const int* __restrict__ rp, const int* __restrict__ agg,
                           const double* __restrict__ pt, int* __restrict__ ci,
                           double* __restrict__ v) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  if (agg[i] >= 0) {
    ci[rp[i]] = agg[i];
    v[rp[i]] = pt[i];
  }
}

// P = P_tent - omega D^-1 (A P_tent); the pattern of A P_tent contains P_tent's.
// omega = 4 / (3 rho) with rho the level's spectral bound (device value).
__global__ void k_smooth_p(int n, const int* __restrict__ qrp, const int* __restrict__ qci,
                           const double* __restrict__ qv, const double* __restrict__ diag,
                           const int* __restrict__ agg, const double* __restrict__ pt,
                           const double* __restrict__ rho, double* __restrict__ pv) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const double omega = 4.0 / (3.0 * *rho);
  const double dinv = 1.0 / diag[i];
  const int ai = agg[i];
  for (int k = qrp[i]; k < qrp[i + 1]; ++k) {
    double t = (qci[k] == ai) ? pt[i] : 0.0;
    pv[k] = t - omega * (qv[k] * dinv);
  }
}

// ------------------------------------------------------------------ spectral bounds
// Gershgorin bound of D^-1 A: block maxima of sum_j |a_ij| / a_ii
__global__ void k_gershgorin(int n, const int* __restrict__ rp, const double* __restrict__ v,
                             const double* __restrict__ diag, double* __restrict__ part) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  double r = 0.0;
  if (i < n) {
    for (int k = rp[i]; k < rp[i + 1]; ++k) r = r + fabs(v[k]);
    r = r / diag[i];
  }
  r = block_max<kBlock>(r);
  if (threadIdx.x == 0) part[blockIdx.x] = r;
}

// The same from the ELL copy (rows of at most WM off-diagonal entries): every
// load coalesced, the diagonal added in its CSR place, so the sums are those of
// the rows bit for bit (1.7 M rows: 40 us from
// the CSR rows, 29 here).
template <int WM>
__global__ void k_gershgorin_ell(int n, int W, const int* __restrict__ ecol,
                                 const double* __restrict__ ev, const double* __restrict__ diag,
                                 double* __restrict__ part) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  double r = 0.0;
  if (i < n) {
    int c[WM];
    slot_cols<WM>(i, n, W, ecol, c);
    const double d = diag[i], a = fabs(d);
    double v[WM];
#pragma unroll
    for (int k = 0; k < WM; ++k) v[k] = c[k] != i ? fabs(ev[(size_t)k * n + i]) : 0.0;
    bool done = false;
#pragma unroll
    for (int k = 0; k < WM; ++k) {
      if (c[k] == i) continue;
      if (!done && c[k] > i) {
        r = r + a;
        done = true;
      }
      r = r + v[k];
    }
    if (!done) r = r + a;
    r = r / d;
  }
  r = block_max<kBlock>(r);
  if (threadIdx.x == 0) part[blockIdx.x] = r;
}

__global__ void __launch_bounds__(kBlock) k_max_partials(const double* __restrict__ part, int g,
                                                         double* __restrict__ out) {
  double m = 0.0;
  for (int b = threadIdx.x; b < g; b += kBlock) m = fmax(m, part[b]);
  m = block_max<kBlock>(m);
  if (threadIdx.x == 0) *out = m;
}

template <int LPR>
__global__ void __launch_bounds__(kBlock) k_diag(int n, const int* __restrict__ rp,
                                                 const int* __restrict__ ci,
                                                 const double* __restrict__ v,
                                                 double* __restrict__ diag, int* __restrict__ flag) {
  const int i = (blockIdx.x * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  double d = 0.0;  // only the lane holding the diagonal adds a nonzero term
  if (i < n)
    for (int k = rp[i] + lane; k < rp[i + 1]; k += LPR)
      if (ci[k] == i) d = v[k];
  d = group_sum<LPR>(d);
  if (i < n && lane == 0) {
    diag[i] = d;
    if (!(d > 0.0)) atomicOr(flag, SE_DIAG);
  }
}

// ------------------------------------------------------------------ sparse products
__device__ __forceinline__ uint32_t slot_hash(int key) { return fmix32((uint32_t)key); }

// Products per row of C = A B: the summed lengths of the rows of B that row
// i of A selects (clipped at 2^30).
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_spgemm_bound(int n, const int* __restrict__ arp,
                                                         const int* __restrict__ aci,
                                                         const int* __restrict__ brp,
                                                         int* __restrict__ prod) {
  const int i = (blockIdx.x * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  long long s = 0;
  if (i < n)
    for (int a = arp[i] + lane; a < arp[i + 1]; a += LPR) s += brp[aci[a] + 1] - brp[aci[a]];
  s = group_sum<LPR>(s);
  if (i < n && lane == 0) prod[i] = s > (1 << 30) ? (1 << 30) : (int)s;
}

// Between a wavefront's own LDS writes and its other lanes' reads of them: the
// operations complete in order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// *p += y in LDS without a result (one operation, no wait)
__device__ __forceinline__ void lds_add(double* p, double y) {
  (void)__hip_atomic_fetch_add(p, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

enum SpMode { SP_COUNT = 0, SP_FILL = 1, SP_DENSE = 2, SP_BITS = 3 };
constexpr int kSpBatch = 4;        // entries of A whose loads are issued together
constexpr int kSpDenseWidth = 512; // widest C accumulated with one slot per column

// Row-parallel C = A B.  Row i of C belongs to W sub-groups of LPR lanes;
// sub-group w walks its contiguous run of row i of A in ascending order and
// scatters the products with each selected row of B into its own value
// array.  The lanes of a sub-group hold distinct columns of that row of B
// and a wavefront's LDS operations complete in issue order, so the products
// reaching one slot from one sub-group are added in entry order with no
// barrier; the sub-groups' arrays are then added in the order w = 0..W-1.
// The result therefore depends only on W, never on timing.  Column slots are
// shared by the row's sub-groups:
//   SP_COUNT  open-addressing hash of column ids (H slots, a power of two);
//             counts[i] = distinct columns of the row;
//   SP_FILL   the same hash; the row is written to C at off[i], sorted by
//             column (rank among the row's columns);
//   SP_DENSE  slot = column (H >= width); the row is written in column order
//             to the scratch row at i stride; counts[i] = entries written;
//   SP_BITS   a bit per column of C in H 32-bit words (no probing); counts[i]
//             = bits set, the row's distinct columns as with SP_COUNT.
// The block holds blockDim / (LPR W) rows; LDS is sized by the host.
template <int LPR, int MODE>
__global__ void __launch_bounds__(1024) k_spgemm_rows(
    int n, int W, int H, const int* __restrict__ arp, const int* __restrict__ aci,
    const double* __restrict__ av, const int* __restrict__ brp, const int* __restrict__ bci,
    const double* __restrict__ bv, const int* __restrict__ off, int stride,
    int* __restrict__ counts, int* __restrict__ cci, double* __restrict__ cv,
    int* __restrict__ flag) {
  extern __shared__ double smem[];
  const int per_row = LPR * W;
  const int rpb = blockDim.x / per_row;
  const int rl = threadIdx.x / per_row, tr = threadIdx.x % per_row;
  const int w = tr / LPR, lane = tr % LPR;
  const int i = blockIdx.x * rpb + rl;
  const bool numeric = MODE == SP_FILL || MODE == SP_DENSE;
  double* vals = smem + (size_t)rl * W * H;  // [W][H] of this row
  int* ibase = reinterpret_cast<int*>(smem + (numeric ? (size_t)rpb * W * H : 0));
  int* keys = ibase + (size_t)rl * H;
  // SP_FILL: the row's occupied slots and their columns, at most H / 2 each
  int* list = ibase + (size_t)rpb * H + (size_t)rl * H;
  int* ckey = list + H / 2;
  int* cnt = ibase + (size_t)(MODE == SP_FILL ? 2 : 1) * rpb * H;
  for (int q = tr; q < H; q += per_row) {
    keys[q] = MODE == SP_BITS ? 0 : -1;
    if (numeric)
      for (int v = 0; v < W; ++v) vals[(size_t)v * H + q] = 0.0;
  }
  if (MODE == SP_DENSE) {
    for (int q = tr; q < per_row / kWave + 1; q += per_row) cnt[rl * (per_row / kWave + 1) + q] = 0;
  } else if (tr == 0) {
    cnt[rl] = 0;
  }
  __syncthreads();

  bool overflow = false;
  auto insert = [&](int key, double y) {
    int q;
    if (MODE == SP_BITS) {
      atomicOr(reinterpret_cast<unsigned*>(keys) + (key >> 5), 1u << (key & 31));
      return;
    }
    if (MODE == SP_DENSE) {
      q = key;
      keys[q] = key;
    } else {
      q = (int)(slot_hash(key) & (uint32_t)(H - 1));
      int probes = 0;
      while (true) {
        const int prev = atomicCAS(&keys[q], -1, key);
        if (prev == -1) {
          if (MODE == SP_COUNT) atomicAdd(&cnt[rl], 1);
          break;
        }
        if (prev == key) break;
        q = (q + 1) & (H - 1);
        if (++probes >= H) { overflow = true; return; }
      }
    }
    if (numeric) vals[(size_t)w * H + q] += y;
  };

  if (i < n) {
    const int a0 = arp[i], a1 = arp[i + 1];
    const int chunk = (a1 - a0 + W - 1) / W;
    const int lo = a0 + w * chunk, hi = min(a1, lo + chunk);
    for (int e = lo; e < hi; e += kSpBatch) {
      int kk[kSpBatch], bb[kSpBatch], be[kSpBatch];
      double xa[kSpBatch], yy[kSpBatch];
#pragma unroll
      for (int u = 0; u < kSpBatch; ++u) {
        kk[u] = -1;
        bb[u] = 0;
        be[u] = 0;
        xa[u] = 0.0;
        yy[u] = 0.0;
        if (e + u < hi) {
          const int j = aci[e + u];
          bb[u] = brp[j];
          be[u] = brp[j + 1];
          if (numeric) xa[u] = av[e + u];
          const int b = bb[u] + lane;
          if (b < be[u]) {
            kk[u] = bci[b];
            if (numeric) yy[u] = xa[u] * bv[b];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kSpBatch; ++u) {
        if (kk[u] >= 0) insert(kk[u], yy[u]);
        for (int b = bb[u] + lane + LPR; b < be[u]; b += LPR)
          insert(bci[b], numeric ? xa[u] * bv[b] : 0.0);
      }
    }
  }
  if (overflow) atomicOr(flag, 1);
  __syncthreads();

  if (MODE == SP_BITS) {
    int c = 0;
    for (int q = tr; q < H; q += per_row) c += __popc((unsigned)keys[q]);
    atomicAdd(&cnt[rl], c);
    __syncthreads();
    if (i < n && tr == 0) counts[i] = cnt[rl];
    return;
  }
  if (MODE == SP_COUNT) {
    if (i < n && tr == 0) counts[i] = cnt[rl];
    return;
  }
  if (MODE == SP_FILL) {
    for (int q = tr; q < H; q += per_row) {
      const int key = keys[q];
      if (key != -1) {
        double v = vals[q];
        for (int u = 1; u < W; ++u) v += vals[(size_t)u * H + q];
        vals[q] = v;
        const int p = atomicAdd(&cnt[rl], 1);
        list[p] = q;
        ckey[p] = key;
      }
    }
    __syncthreads();
    if (i >= n) return;
    const int u = cnt[rl], base = off[i];
    for (int p = tr; p < u; p += per_row) {
      const int key = ckey[p];
      int rank = 0;
      for (int q = 0; q < u; ++q) rank += ckey[q] < key ? 1 : 0;
      cci[base + rank] = key;
      cv[base + rank] = vals[list[p]];
    }
    return;
  }
  // SP_DENSE: thread tr owns the contiguous slots [s0, s1); an exclusive scan
  // of the owned counts over the row's threads gives each its output offset.
  const int per = (H + per_row - 1) / per_row;
  const int s0 = min(H, tr * per), s1 = min(H, s0 + per);
  int c = 0;
  for (int q = s0; q < s1; ++q) c += keys[q] != -1 ? 1 : 0;
  const int width = per_row < kWave ? per_row : kWave;
  int inc = c;
  const int wl = tr % width;
  for (int o = 1; o < width; o <<= 1) {
    const int t = __shfl_up(inc, o, width);
    if (wl >= o) inc += t;
  }
  int* wtot = cnt + rl * (per_row / kWave + 1);
  if (per_row > kWave) {
    if (wl == width - 1) wtot[tr / kWave] = inc;
    __syncthreads();
    int before = 0;
    for (int q = 0; q < tr / kWave; ++q) before += wtot[q];
    inc += before;
  }
  if (i >= n) return;
  int pos = i * stride + inc - c;
  for (int q = s0; q < s1; ++q) {
    if (keys[q] != -1) {
      double v = vals[q];
      for (int u = 1; u < W; ++u) v += vals[(size_t)u * H + q];
      cci[pos] = q;
      cv[pos] = v;
      ++pos;
    }
  }
  if (tr == per_row - 1) counts[i] = inc;
}

// C = A B in one pass, W wavefronts per row (1 or kSpWaves).  A wavefront's
// products go to value slots found by a hash in LDS (H = 2 cap slots, keys
// shared by the row's wavefronts): 64 / LPR entries of A's row at a time, LPR
// lanes across the selected row of B.  Sub-groups that meet in a column would
// add in an order of their own, so the adds are issued one sub-group after
// another; they return nothing, so nothing waits for them, and a wavefront's LDS
// operations complete in issue order.  So a column is summed from 0 in an order
// that A's and B's rows fix, whatever the timing: of each 64 / LPR entries of A's
// row the first LPR columns of every selected row, in entry order, then the next
// LPR of every one, and so on (the entry order itself where no selected row is
// longer than LPR); then the wavefronts' sums in theirs.  The row is written
// sorted by column to the scratch row at i cap, and counts[i] = its length; a
// row of more than cap columns sets *over and the host takes the two passes of k_spgemm_rows (a wavefront stops after its first column without
// a slot: for every later product it would probe all of a full table, which made
// the set-up of 100^3 cells with a shift, 22.5 k rows of 279 columns in 256
// slots, 14.7 ms; 8.5 so, and 7.2 where the host foresees it).
// It replaces a counting pass with a table of the product bound and a filling
// one with a value array per sub-group, whose initialisation, merging and
// probing were most of their LDS traffic.  R (A P) of a 128^3 system's finest
// level (133 k rows of 390 products) took 258 + 447 us and takes 293 + 36 with
// the compaction, the next level's A P (210 products) 107 + 403 and takes 221 +
// 19; the 128^3 set-up went from 5.14 to 4.35 ms.  What is left is LDS (41% of
// the cycles) and vector instructions (about 60%) of the claims and the adds.
constexpr int kSpWaves = 4;  // wavefronts per block
// Scratch columns per row where fewer are not known to do.  Rows of 3D meshes'
// coarse operators stay below 100 up to some 10^4 rows; 128 rather than 256
// keeps eight blocks per compute unit in LDS.
constexpr int kSpCap = 128, kSpCapFew = 256;
constexpr int kSpFewRows = 16384;
// Entries of scratch (12 bytes each) beyond which the two passes, which need
// none, are taken: 3 GB, about one percent of the device's memory, reached with
// two million coarse rows.  They are also taken where less is not to be had.
constexpr int64_t kSpScratch = int64_t(1) << 28;
// A row of C is a union of rows of B that overlap: in hierarchies of boxes,
// plates and beams its longest row held 1.6 to 4.6 times as many columns as B's
// longest one (R A P of shifted systems' second level 3.6 to 4.6, with rows up to
// 514).  Where kSpUnion times B's longest row passes the scratch row, the pass
// would in all likelihood only be found too short, so the two passes are taken
// at once.
constexpr int kSpUnion = 4;
// Lanes' worth of products above which a row is shared by the block's
// wavefronts: 11.6 k rows of 84 entries x 32 lanes take 151 us with one and 106
// with four, 13.8 k rows of 39 entries x 16 lanes 40 with one and 53 with four.
constexpr int kSpSplit = 1024;

// LDS of one row: W value arrays and the keys of H = 2 cap slots, and the
// staged entries of A, which the list of columns takes over afterwards.
inline __host__ __device__ size_t spgemm_wave_lds(int cap, int W) {
  const size_t list = (size_t)6 * cap, staged = (size_t)W * kWave * 16;
  return (size_t)2 * cap * (8 * W + 4) + (list > staged ? list : staged);
}

template <int LPR, int W>
__global__ void __launch_bounds__(kSpWaves* kWave) k_spgemm_wave(
    int n, int cap, int hshift, const int* __restrict__ arp, const int* __restrict__ aci,
    const double* __restrict__ av, const int* __restrict__ brp, const int* __restrict__ bci,
    const double* __restrict__ bv, int* __restrict__ counts, int* __restrict__ sci,
    double* __restrict__ sv, int* __restrict__ over) {
  extern __shared__ char spw[];
  constexpr int S = kWave / LPR, kRow = W * kWave;  // threads of a row
  const int H = 2 * cap;
  const int row = threadIdx.x / kRow, t = threadIdx.x % kRow, w = t / kWave, lane = t % kWave;
  const int sub = lane / LPR, bl = lane % LPR;
  char* mine = spw + (size_t)row * spgemm_wave_lds(cap, W);
  double* vals = reinterpret_cast<double*>(mine);  // [W][H]
  int* keys = reinterpret_cast<int*>(vals + (size_t)W * H);
  int4* staged = reinterpret_cast<int4*>(keys + H) + w * kWave;
  int* ckey = keys + H;
  unsigned short* slot = reinterpret_cast<unsigned short*>(ckey + cap);
  const int i = xcd_block(blockIdx.x, gridDim.x) * (kSpWaves / W) + row;
  if (i >= n) return;  // whole rows: a row of several wavefronts is a block
  // between LDS writes and other lanes' reads of them
  auto fence = [] {
    if (W > 1) __syncthreads();
    else wave_lds_fence();
  };
  for (int q = t; q < H / 4; q += kRow) reinterpret_cast<int4*>(keys)[q] = make_int4(-1, -1, -1, -1);
  for (int q = t; q < W * H / 2; q += kRow)
    reinterpret_cast<double2*>(vals)[q] = make_double2(0.0, 0.0);
  vals += (size_t)w * H;
  fence();

  bool full = false;
  auto claim = [&](int key) {  // key's slot (key < 0: none)
    int q = (int)(((uint32_t)key * 0x9E3779B1u) >> hshift);
    if (key >= 0) {
      int prev = atomicCAS(&keys[q], -1, key);
      for (int probes = 0; prev != -1 && prev != key; ++probes) {
        if (probes == cap) {
          full = true;
          break;
        }
        q = (q + 1) & (H - 1);
        prev = atomicCAS(&keys[q], -1, key);
      }
    }
    return q;
  };
  auto add = [&](int key, int q, double y) {
#pragma unroll
    for (int g = 0; g < S; ++g)
      if (sub == g && key >= 0) lds_add(&vals[q], y);
  };

  // wavefront w's run of the row's entries
  const int r0 = arp[i], r1 = arp[i + 1], run = (r1 - r0 + W - 1) / W;
  const int a0 = r0 + w * run, a1 = min(r1, a0 + run);
  for (int c0 = a0; c0 < a1; c0 += kWave) {
    const int len = min(kWave, a1 - c0);
    int4 mineA = make_int4(0, 0, 0, 0);  // the selected row's ends, A's value
    if (lane < len) {
      const int j = aci[c0 + lane];
      const double x = av[c0 + lane];
      mineA = make_int4(brp[j], brp[j + 1], __double2loint(x), __double2hiint(x));
    }
    wave_lds_fence();
    staged[lane] = mineA;
    wave_lds_fence();
    for (int e = 0; e < len; e += S * kSpBatch) {
      if (__any(full)) break;
      int b0[kSpBatch], b1[kSpBatch], kk[kSpBatch], qq[kSpBatch];
      double xx[kSpBatch], yy[kSpBatch];
#pragma unroll
      for (int u = 0; u < kSpBatch; ++u) {
        const int src = e + u * S + sub;
        const int4 en = staged[src & (kWave - 1)];
        b0[u] = en.x + bl;
        b1[u] = src < len ? en.y : 0;
        xx[u] = __hiloint2double(en.w, en.z);
        kk[u] = -1;
        yy[u] = 0.0;
        if (b0[u] < b1[u]) {
          kk[u] = bci[b0[u]];
          yy[u] = xx[u] * bv[b0[u]];
        }
      }
#pragma unroll
      for (int u = 0; u < kSpBatch; ++u) qq[u] = claim(kk[u]);
#pragma unroll
      for (int u = 0; u < kSpBatch; ++u) {
        if (e + u * S >= len) break;
        add(kk[u], qq[u], yy[u]);
        for (int b = b0[u] + LPR; __any(b < b1[u]); b += LPR) {
          int key = -1;
          double y = 0.0;
          if (b < b1[u]) {
            key = bci[b];
            y = xx[u] * bv[b];
          }
          const int q = claim(key);
          add(key, q, y);
        }
      }
    }
  }
  if (__any(full) && lane == 0) atomicOr(over, 1);
  fence();
  vals -= (size_t)w * H;

  // every wavefront lists the columns for itself (the last write of equal
  // values stands) and takes its share of them
  int u = 0;
  for (int q = lane; q < H; q += kWave) {
    const int key = keys[q];
    const unsigned long long m = __ballot(key != -1);
    if (key != -1) {
      const int p = u + __popcll(m & ((1ull << lane) - 1));
      if (p < cap) {
        ckey[p] = key;
        slot[p] = (unsigned short)q;
      }
    }
    u += __popcll(m);
  }
  if (t == 0) counts[i] = u;
  if (u > cap) {
    if (t == 0) atomicOr(over, 1);
    return;
  }
  if (lane < ((4 - (u & 3)) & 3)) ckey[u + lane] = INT32_MAX;  // cap is a multiple of 4
  wave_lds_fence();
  const size_t base = (size_t)i * cap;
  for (int p = t; p < u; p += kRow) {
    const int key = ckey[p], q = slot[p];
    double v = vals[q];
#pragma unroll
    for (int k = 1; k < W; ++k) v += vals[(size_t)k * H + q];
    int rank = 0;
    for (int o4 = 0; o4 < u; o4 += 4) {
      const int4 o = *reinterpret_cast<const int4*>(ckey + o4);
      rank += (o.x < key ? 1 : 0) + (o.y < key ? 1 : 0) + (o.z < key ? 1 : 0) + (o.w < key ? 1 : 0);
    }
    sci[base + rank] = key;
    sv[base + rank] = v;
  }
}

// Copy the rows of a product from scratch rows (at i stride) into C.
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_spgemm_compact(int n, int stride,
                                                           const int* __restrict__ crp,
                                                           const int* __restrict__ sci,
                                                           const double* __restrict__ sv,
                                                           int* __restrict__ cci,
                                                           double* __restrict__ cv) {
  const int i = (blockIdx.x * kBlock + threadIdx.x) / LPR, lane = threadIdx.x % LPR;
  if (i >= n) return;
  const int src = i * stride, dst = crp[i], len = crp[i + 1] - dst;
  for (int k = lane; k < len; k += LPR) {
    cci[dst + k] = sci[src + k];
    cv[dst + k] = sv[src + k];
  }
}

// ------------------------------------------------------------------ transpose
// A narrow matrix (at most kNarrowCols columns, such as the prolongator onto
// the coarsest level) is transposed without atomics on its few column
// counters and without sorting: a one-workgroup count, then one workgroup
// per column that collects the column's entries in storage order.
// Every column's workgroup walks all entries twice, while the general path's
// rank sort compares every pair of a column's entries, so which is faster
// depends on columns x entries against the square of the mean column:
//
//   columns x entries     over mean^2     narrow, us   general, us
//   4.3 M (97 x 44 k)           21             56          126
//   19 M (169 x 115 k)          42            105          271
//   50 M (287 x 175 k)         135            147          243
//   288 M (487 x 591 k)        195            461          809
//   194 M (546 x 355 k)        457            409          273
//   10.6 M (270 x 39 k)        503             42           27
//   31 M (455 x 69 k)        1,370             67           28
//
// (kernel times on prolongators of boxes from 12^3 to 128^3, beams and plates,
// with and without a shift; a line between 195 and 281 parts them all).  Up to
// kNarrowWork columns x entries the narrow path's fewer launches make up for
// what its kernels lose.
constexpr int kNarrowCols = 1024;
constexpr int64_t kNarrowWork = int64_t(8) << 20;
constexpr int64_t kNarrowRatio = 256;
inline bool narrow_pays(int64_t cols, int64_t nnz) {
  if (cols <= 0 || nnz <= 0 || cols > kNarrowCols) return false;
  // cols nnz / (nnz / cols)^2 = cols^3 / nnz
  return cols * nnz <= kNarrowWork || cols * cols * cols <= kNarrowRatio * nnz;
}
constexpr int kNarrowU = 8;  // entries per lane whose loads are issued together

// Column counts in LDS, then T's row pointers trp[0..m] (exclusive scan over
// the columns) and its longest row *rmax.  One workgroup of 1024 threads.
__global__ void __launch_bounds__(1024) k_narrow_count(int64_t nnz, int m,
                                                       const int* __restrict__ ci,
                                                       int* __restrict__ trp,
                                                       int* __restrict__ rmax) {
  __shared__ int h[kNarrowCols];
  __shared__ int wsum[1024 / kWave];
  __shared__ int hmax;
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  h[t] = 0;
  if (t == 0) hmax = 0;
  __syncthreads();
  for (int64_t k0 = t; k0 < nnz; k0 += 1024 * kNarrowU) {
    int c[kNarrowU];
#pragma unroll
    for (int u = 0; u < kNarrowU; ++u) {
      const int64_t k = k0 + (int64_t)u * 1024;
      c[u] = k < nnz ? ci[k] : -1;
    }
#pragma unroll
    for (int u = 0; u < kNarrowU; ++u)
      if (c[u] >= 0) atomicAdd(&h[c[u]], 1);
  }
  __syncthreads();
  const int v = t < m ? h[t] : 0;
  atomicMax(&hmax, v);
  int inc = v;
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(inc, o, kWave);
    if (lane >= o) inc += u;
  }
  if (lane == kWave - 1) wsum[w] = inc;
  __syncthreads();
  int before = 0;
  for (int q = 0; q < w; ++q) before += wsum[q];
  if (t < m) trp[t] = before + inc - v;
  if (t == m - 1) trp[m] = before + inc;
  if (t == 0) *rmax = hmax;
}

// rowid[k] = the row of entry k.
__global__ void k_row_ids(int n, const int* __restrict__ rp, int* __restrict__ rowid) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n)
    for (int k = rp[i]; k < rp[i + 1]; ++k) rowid[k] = i;
}

// Row J = blockIdx.x of T: wave w of the workgroup takes the w-th run of A's
// entries in storage order, counts those in column J (ballots), and after
// the counts of the earlier runs writes them in order.  Storage order is
// ascending row, so T's rows come out sorted.
__global__ void __launch_bounds__(1024) k_narrow_fill(int64_t nnz, const int* __restrict__ ci,
                                                      const double* __restrict__ v,
                                                      const int* __restrict__ rowid,
                                                      const int* __restrict__ trp,
                                                      int* __restrict__ tci,
                                                      double* __restrict__ tv) {
  __shared__ int wcnt[1024 / kWave];
  const int J = blockIdx.x;
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  constexpr int nw = 1024 / kWave, step = kWave * kNarrowU;
  const int64_t chunk = (nnz + nw - 1) / nw;
  const int64_t k0 = min(nnz, (int64_t)w * chunk), k1 = min(nnz, k0 + chunk);
  const unsigned long long below = (1ull << lane) - 1ull;
  int c = 0;
  for (int64_t base = k0; base < k1; base += step) {
    bool hit[kNarrowU];
#pragma unroll
    for (int u = 0; u < kNarrowU; ++u) {
      const int64_t k = base + (int64_t)u * kWave + lane;
      hit[u] = k < k1 && ci[k] == J;
    }
#pragma unroll
    for (int u = 0; u < kNarrowU; ++u) c += __popcll(__ballot(hit[u]));
  }
  if (lane == 0) wcnt[w] = c;
  __syncthreads();
  int pos = trp[J];
  for (int q = 0; q < w; ++q) pos += wcnt[q];
  for (int64_t base = k0; base < k1; base += step) {
    bool hit[kNarrowU];
#pragma unroll
    for (int u = 0; u < kNarrowU; ++u) {
      const int64_t k = base + (int64_t)u * kWave + lane;
      hit[u] = k < k1 && ci[k] == J;
    }
#pragma unroll
    for (int u = 0; u < kNarrowU; ++u) {
      const unsigned long long mask = __ballot(hit[u]);
      if (hit[u]) {
        const int64_t k = base + (int64_t)u * kWave + lane;
        const int p = pos + __popcll(mask & below);
        tci[p] = rowid[k];
        tv[p] = v[k];
      }
      pos += __popcll(mask);
    }
  }
}

// Column counts of a CSR, and for every entry its place among its column's
// (with the aggregate of each node for column: member counts and places; a
// negative column is none).
// Consecutive entries belong to neighbouring rows and share columns, and
// device-scope atomics, not the loads, bound a pass with one per entry: a block
// counts its kSlotChunk entries in an LDS hash of their columns and then takes
// the places of each column at once.  The filling pass needs no atomics after
// that.  Against atomics once per column and wavefront in both passes: 5.2 M
// entries in 133 k columns 51 + 117 us and now 45 + 55, 92 k entries in 632
// columns 10 + 31 and 8 + 4 (the 64^3 set-up 1,490 -> 1,420 us).
constexpr int kSlotItems = 8, kSlotChunk = kBlock * kSlotItems;

__global__ void __launch_bounds__(kBlock) k_col_slots(int64_t nnz, const int* __restrict__ ci,
                                                      int* __restrict__ cnt,
                                                      int* __restrict__ pos) {
  __shared__ int keys[kSlotChunk], num[kSlotChunk];  // at most a column per entry
  const int64_t k0 = (int64_t)blockIdx.x * kSlotChunk;
  int c[kSlotItems], at[kSlotItems], mine[kSlotItems];
#pragma unroll
  for (int u = 0; u < kSlotItems; ++u) {
    const int64_t k = k0 + u * kBlock + threadIdx.x;
    c[u] = k < nnz ? ci[k] : -1;
  }
#pragma unroll
  for (int u = 0; u < kSlotItems; ++u) {
    keys[u * kBlock + threadIdx.x] = -1;
    num[u * kBlock + threadIdx.x] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSlotItems; ++u) {
    if (c[u] < 0) continue;
    int q = (int)(((uint32_t)c[u] * 0x9E3779B1u) >> 21);
    for (;;) {
      const int prev = atomicCAS(&keys[q], -1, c[u]);
      if (prev == -1 || prev == c[u]) break;
      q = (q + 1) & (kSlotChunk - 1);
    }
    at[u] = q;
    mine[u] = atomicAdd(&num[q], 1);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSlotItems; ++u) {
    const int q = u * kBlock + threadIdx.x;
    if (keys[q] >= 0) num[q] = atomicAdd(&cnt[keys[q]], num[q]);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSlotItems; ++u)
    if (c[u] >= 0) pos[k0 + u * kBlock + threadIdx.x] = num[at[u]] + mine[u];
}

// Each entry (i, c) of row i to its place in row c of the transpose (the order
// within a row is fixed afterwards by k_rank_rows).
template <int LPR>
__global__ void __launch_bounds__(kBlock) k_transpose_fill(
    int n, const int* __restrict__ rp, const int* __restrict__ ci, const double* __restrict__ v,
    const int* __restrict__ trp, const int* __restrict__ pos, int* __restrict__ tci,
    double* __restrict__ tv) {
  const int i = (xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x) / LPR;
  const int lane = threadIdx.x % LPR;
  if (i >= n) return;
  for (int k = rp[i] + lane; k < rp[i + 1]; k += LPR) {
    const int p = trp[ci[k]] + pos[k];
    tci[p] = i;
    tv[p] = v[k];
  }
}

// Sort every row of an unsorted CSR by column into (ci, v): one 64-lane
// workgroup per row; each entry's destination is the number of smaller keys
// in its row (keys are distinct within a row).  Rows up to kRankStage
// entries are compared from LDS.  (Four rows per workgroup was slower: the
// barrier waits for the block's longest row.)
constexpr int kRankStage = 2048;
__global__ void __launch_bounds__(kWave) k_rank_rows(const int* __restrict__ rp,
                                                     const int* __restrict__ uci,
                                                     const double* __restrict__ uv,
                                                     int* __restrict__ ci, double* __restrict__ v) {
  __shared__ int sk[kRankStage];
  const int i = blockIdx.x;
  const int b = rp[i], e = rp[i + 1], len = e - b;
  const bool staged = len <= kRankStage;
  if (staged)
    for (int p = threadIdx.x; p < len; p += kWave) sk[p] = uci[b + p];
  __syncthreads();
  for (int p = threadIdx.x; p < len; p += kWave) {
    const int key = staged ? sk[p] : uci[b + p];
    int rank = 0;
    if (staged)
      for (int q = 0; q < len; ++q) rank += sk[q] < key ? 1 : 0;
    else
      for (int q = b; q < e; ++q) rank += uci[q] < key ? 1 : 0;
    ci[b + rank] = key;
    v[b + rank] = uv[b + p];
  }
}

// ------------------------------------------------------------------ dense coarsest
// Explicit inverse of the SPD coarsest matrix by Gauss-Jordan elimination
// without pivoting (pivots of an SPD matrix are positive): at step k the
// pivot row is divided by the pivot with a_kk replaced by 1, and every other
// row i gets a_ij -= f_i a_kj with a_ik replaced by 0 (f the pivot column),
// which leaves A^-1 in place of A.  Up to kDenseBlk rows one workgroup does
// it from the n x n row-major array G = A (k_dense_inverse_blk);
// larger levels take the blocked form over many workgroups (k_ginv_*).
constexpr int kDenseBlk = 128;

// The elimination for n <= 128 by 4 x 4 blocks: thread t owns the block
// of rows 4 (t / 32) .. +3 and columns 4 (t mod 32) .. +3 of the 128 x 128
// cover, padded with the identity past n (the padding stays decoupled).
// Block step K (pivots 4K .. 4K+3) is the block form of the steps above: with
// D = A_KK, C_I = A_IK and R_J = A_KJ,
//   A_KK <- D^-1,  A_KJ <- D^-1 R_J,  A_IK <- -C_I D^-1,
//   A_IJ <- A_IJ - C_I (D^-1 R_J).
// The owner of A_KK inverts it in registers by the scalar steps (its four
// pivots are the elimination's pivots 4K .. 4K+3, each checked > 0).  D^-1,
// the old block column and the new block row pass through LDS,
// double-buffered, so a block step takes two barriers instead of the four
// of four scalar steps.
__global__ void __launch_bounds__(1024) k_dense_inverse_blk(int n, const double* __restrict__ Gm,
                                                            double* __restrict__ Ainv,
                                                            int* __restrict__ flag) {
  constexpr int B = 4;
  __shared__ double dinv[2][B][B];
  __shared__ double cpan[2][32 * B][B];
  __shared__ double rpan[2][B][32 * B];
  const int t = threadIdx.x;
  const int I = t / 32, J = t % 32, i0 = I * B, j0 = J * B;
  double a[B][B];
#pragma unroll
  for (int r = 0; r < B; ++r)
#pragma unroll
    for (int c = 0; c < B; ++c) {
      const int i = i0 + r, j = j0 + c;
      a[r][c] = (i < n && j < n) ? Gm[(size_t)i * n + j] : (i == j ? 1.0 : 0.0);
    }
  const int nb = (n + B - 1) / B;
  for (int K = 0; K < nb; ++K) {
    const int bf = K & 1;
    if (I == K && J == K) {
#pragma unroll
      for (int k = 0; k < B; ++k) {
        double piv = a[k][k];
        if (!(piv > 0.0)) {
          atomicOr(flag, SE_DENSE);
          piv = 1.0;
        }
        const double inv = 1.0 / piv;
        double rk[B];
#pragma unroll
        for (int c = 0; c < B; ++c) rk[c] = (c == k ? 1.0 : a[k][c]) * inv;
#pragma unroll
        for (int r = 0; r < B; ++r) {
          if (r == k) continue;
          const double f = a[r][k];
#pragma unroll
          for (int c = 0; c < B; ++c) a[r][c] = (c == k ? 0.0 : a[r][c]) - f * rk[c];
        }
#pragma unroll
        for (int c = 0; c < B; ++c) a[k][c] = rk[c];
      }
#pragma unroll
      for (int r = 0; r < B; ++r)
#pragma unroll
        for (int c = 0; c < B; ++c) dinv[bf][r][c] = a[r][c];
    }
    if (J == K && I != K) {
#pragma unroll
      for (int r = 0; r < B; ++r)
#pragma unroll
        for (int c = 0; c < B; ++c) cpan[bf][i0 + r][c] = a[r][c];
    }
    __syncthreads();
    if (I == K && J != K) {  // the block row: D^-1 R_J
      double nr[B][B];
#pragma unroll
      for (int r = 0; r < B; ++r)
#pragma unroll
        for (int c = 0; c < B; ++c) {
          double s = 0.0;
#pragma unroll
          for (int m = 0; m < B; ++m) s = fma(dinv[bf][r][m], a[m][c], s);
          nr[r][c] = s;
        }
#pragma unroll
      for (int r = 0; r < B; ++r)
#pragma unroll
        for (int c = 0; c < B; ++c) {
          a[r][c] = nr[r][c];
          rpan[bf][r][j0 + c] = nr[r][c];
        }
    }
    __syncthreads();
    if (I != K) {
      double f[B][B];
#pragma unroll
      for (int r = 0; r < B; ++r)
#pragma unroll
        for (int m = 0; m < B; ++m) f[r][m] = cpan[bf][i0 + r][m];
      if (J == K) {  // the block column: -C_I D^-1
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
          for (int c = 0; c < B; ++c) {
            double s = 0.0;
#pragma unroll
            for (int m = 0; m < B; ++m) s = fma(f[r][m], dinv[bf][m][c], s);
            a[r][c] = -s;
          }
      } else {
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
          for (int c = 0; c < B; ++c) {
            double s = a[r][c];
#pragma unroll
            for (int m = 0; m < B; ++m) s = fma(-f[r][m], rpan[bf][m][j0 + c], s);
            a[r][c] = s;
          }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < B; ++r)
#pragma unroll
    for (int c = 0; c < B; ++c)
      if (i0 + r < n && j0 + c < n) Ainv[(size_t)(i0 + r) * n + j0 + c] = a[r][c];
}

// ---- blocked Gauss-Jordan over several workgroups (coarsest levels of 257
// to 1024 rows).  The SPD matrix is padded with the identity to N = 32 nb
// rows and eliminated by 32 x 32 blocks: at block step K the diagonal block
// D = G[K][K] is inverted by the scalar steps (its 32 pivots are the
// elimination's pivots 32K .. 32K+31, each checked > 0), then every block is
// rewritten from the old matrix into the other buffer:
//   G'[K][K] = D^-1,  G'[K][J] = D^-1 G[K][J],  G'[I][K] = -G[I][K] D^-1,
//   G'[I][J] = G[I][J] - G[I][K] (D^-1 G[K][J]).
// Reading only the old matrix, the blocks need no ordering among themselves.

//
// One dispatch per block step: the products run on the FP64 matrix cores (one
// 16 x 16 quadrant per wave), and the workgroup that rewrites the next
// diagonal block inverts it at once for the next step.  A 279-row level takes
// 11 dispatches and 120 us; with the diagonal block inverted by a dispatch of
// its own (two barriers per pivot) and the products added up from LDS it took
// 21 and 225.
typedef double double4_t __attribute__((ext_vector_type(4)));
constexpr int kGinvB = 32, kGinvPitch = kGinvB + 4;

// Inverts the 32 x 32 block held by a workgroup of 256 threads, thread t with
// rows t / 32 + 8 q of column t mod 32.  Two pivots per step, by the inverse
// of their 2 x 2 block: what a step costs is its chain (the pivots' rows and
// columns through LDS and a barrier, a division, two products), not its
// arithmetic.
__device__ __forceinline__ void invert_block(double (&d)[4], int* __restrict__ flag) {
  __shared__ double row[2][2][kGinvB], col[2][2][kGinvB];
  const int c = threadIdx.x % kGinvB, r0 = threadIdx.x / kGinvB;
  auto publish = [&](int k) {
    const int buf = (k >> 1) & 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = r0 + 8 * q;
      if ((r & ~1) == k) row[buf][r & 1][c] = d[q];
      if ((c & ~1) == k) col[buf][c & 1][r] = d[q];
    }
    __syncthreads();
  };
  publish(0);
  for (int k = 0; k < kGinvB; k += 2) {
    const int buf = (k >> 1) & 1;
    const double p00 = row[buf][0][k], p01 = row[buf][0][k + 1];
    const double p10 = row[buf][1][k], p11 = row[buf][1][k + 1];
    const double x0 = row[buf][0][c], x1 = row[buf][1][c];
    double f0[4], f1[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f0[q] = col[buf][0][r0 + 8 * q];
      f1[q] = col[buf][1][r0 + 8 * q];
    }
    double det = fma(p00, p11, -(p01 * p10));
    if (!(p00 > 0.0 && det > 0.0)) {  // both pivots of the elimination are positive
      if (threadIdx.x == 0) atomicOr(flag, SE_DENSE);
      det = 1.0;
    }
    const double inv = 1.0 / det;
    // this column of the pivots' rows of [P | I], then of P^-1 times them
    const double u0 = c == k ? 1.0 : c == k + 1 ? 0.0 : x0;
    const double u1 = c == k ? 0.0 : c == k + 1 ? 1.0 : x1;
    const double n0 = (p11 * u0 - p01 * u1) * inv, n1 = (p00 * u1 - p10 * u0) * inv;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = r0 + 8 * q;
      const double rest = ((c & ~1) == k ? 0.0 : d[q]) - (f0[q] * n0 + f1[q] * n1);
      d[q] = r == k ? n0 : r == k + 1 ? n1 : rest;
    }
    if (k + 2 < kGinvB) publish(k + 2);
  }
}

// Dinv = the inverse of G's first diagonal block (N x N row-major G).
__global__ void __launch_bounds__(256) k_ginv_first(int N, const double* __restrict__ G,
                                                    double* __restrict__ Dinv,
                                                    int* __restrict__ flag) {
  const int c = threadIdx.x % kGinvB, r0 = threadIdx.x / kGinvB;
  double d[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) d[q] = G[(size_t)(r0 + 8 * q) * N + c];
  invert_block(d, flag);
#pragma unroll
  for (int q = 0; q < 4; ++q) Dinv[(r0 + 8 * q) * kGinvB + c] = d[q];
}

// The wave's quadrant of X Y (32 x 32 operands in LDS).  Operands and result
// of v_mfma_f64_16x16x4f64: lane l holds X[l % 16][l / 16], Y[l / 16][l % 16]
// and, as accumulator r, (X Y)[l / 16 + 4 r][l % 16].
__device__ __forceinline__ double4_t block_product(const double (&X)[kGinvB][kGinvPitch],
                                                   const double (&Y)[kGinvB][kGinvPitch], int r0,
                                                   int c0) {
  const int i = threadIdx.x % 16, kq = (threadIdx.x % kWave) / 16;
  double4_t acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kGinvB; k += 4)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[r0 + i][k + kq], Y[k + kq][c0 + i], acc, 0, 0, 0);
  return acc;
}

// Block step K over all blocks: workgroup (J, I) writes block (I, J) of Gn;
// the one of block (K + 1, K + 1) also leaves that block's inverse in next.
__global__ void __launch_bounds__(256) k_ginv_step(int N, const double* __restrict__ G,
                                                   const double* __restrict__ Dinv, int K,
                                                   double* __restrict__ Gn,
                                                   double* __restrict__ next,
                                                   int* __restrict__ flag) {
  __shared__ double Ds[kGinvB][kGinvPitch], Rs[kGinvB][kGinvPitch], Cs[kGinvB][kGinvPitch],
      Ts[kGinvB][kGinvPitch];
  const int I = blockIdx.y, J = blockIdx.x;
  const int c = threadIdx.x % kGinvB, r0 = threadIdx.x / kGinvB;
  const size_t row = (size_t)I * kGinvB, col = (size_t)J * kGinvB, kk = (size_t)K * kGinvB;
  if (I == K && J == K) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      Gn[(row + r0 + 8 * q) * N + col + c] = Dinv[(r0 + 8 * q) * kGinvB + c];
    return;
  }
  double g[4];  // the block itself, requested with the operands
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + 8 * q;
    Ds[r][c] = Dinv[r * kGinvB + c];
    if (J != K) Rs[r][c] = G[(kk + r) * N + col + c];
    if (I != K) Cs[r][c] = G[(row + r) * N + kk + c];
    g[q] = I != K && J != K ? G[(row + r) * N + col + c] : 0.0;
  }
  __syncthreads();
  const int wv = threadIdx.x / kWave, qr = 16 * (wv / 2), qc = 16 * (wv % 2);
  const int ar = qr + (threadIdx.x % kWave) / 16, ac = qc + threadIdx.x % 16;  // acc 0's place
  // D^-1 R for the blocks right and left of the diagonal one, -C D^-1 for
  // those above and below it, C (D^-1 R) elsewhere
  double4_t acc = J == K ? block_product(Cs, Ds, qr, qc) : block_product(Ds, Rs, qr, qc);
  if (I == K || J == K) {
    const double sign = J == K ? -1.0 : 1.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) Gn[(row + ar + 4 * r) * N + col + ac] = sign * acc[r];
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) Ts[ar + 4 * r][ac] = acc[r];
  __syncthreads();
  acc = block_product(Cs, Ts, qr, qc);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) Ts[ar + 4 * r][ac] = acc[r];  // back to the loads' layout
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    g[q] = g[q] - Ts[r0 + 8 * q][c];
    Gn[(row + r0 + 8 * q) * N + col + c] = g[q];
  }
  if (I == K + 1 && J == K + 1) {
    invert_block(g, flag);
#pragma unroll
    for (int q = 0; q < 4; ++q) next[(r0 + 8 * q) * kGinvB + c] = g[q];
  }
}

// G = A padded with the identity to N x N, row-major: one workgroup per row,
// assembled in LDS (N <= kDenseMax).
__global__ void __launch_bounds__(kBlock) k_densify(int n, int N, const int* __restrict__ rp,
                                                    const int* __restrict__ ci,
                                                    const double* __restrict__ v,
                                                    double* __restrict__ G) {
  __shared__ double rowv[kDenseMax];
  const int i = blockIdx.x;
  for (int j = threadIdx.x; j < N; j += kBlock) rowv[j] = i >= n && j == i ? 1.0 : 0.0;
  __syncthreads();
  if (i < n)
    for (int k = rp[i] + threadIdx.x; k < rp[i + 1]; k += kBlock) rowv[ci[k]] = v[k];
  __syncthreads();
  for (int j = threadIdx.x; j < N; j += kBlock) G[(size_t)i * N + j] = rowv[j];
}

// ------------------------------------------------------------------ host helpers
// Launch a lane-grouped row kernel K<LPR> over `rows` rows.
#define PPE_ROWS(LPR_, K, rows, ...)                                                         \
  do {                                                                                       \
    const int lpr_ = (LPR_);                                                                 \
    const int g_ = grid_for((int64_t)(rows) * lpr_);                                         \
    switch (lpr_) {                                                                          \
      case 1: hipLaunchKernelGGL(K<1>, dim3(g_), dim3(kBlock), 0, s->stream, __VA_ARGS__); break;   \
      case 2: hipLaunchKernelGGL(K<2>, dim3(g_), dim3(kBlock), 0, s->stream, __VA_ARGS__); break;   \
      case 4: hipLaunchKernelGGL(K<4>, dim3(g_), dim3(kBlock), 0, s->stream, __VA_ARGS__); break;   \
      case 8: hipLaunchKernelGGL(K<8>, dim3(g_), dim3(kBlock), 0, s->stream, __VA_ARGS__); break;   \
      case 16: hipLaunchKernelGGL(K<16>, dim3(g_), dim3(kBlock), 0, s->stream, __VA_ARGS__); break; \
      case 32: hipLaunchKernelGGL(K<32>, dim3(g_), dim3(kBlock), 0, s->stream, __VA_ARGS__); break; \
      default: hipLaunchKernelGGL(K<64>, dim3(g_), dim3(kBlock), 0, s->stream, __VA_ARGS__); break; \
    }                                                                                        \
    PPE_LAUNCH_CHECK();                                                                      \
  } while (0)
// Lanes per row of the aggregation kernels (strength, the MIS-2 rounds and
// the two joining passes): the power of two from 1 to 64 nearest to half the
// mean row length.  Their results are maxima and per-entry tests, so they do
// not depend on it.
static int agg_lanes(const Csr& A) {
  const double target = (A.n ? (double)A.nnz / A.n : 1.0) / 2.0;
  int best = 1;
  for (int c = 2; c <= 64; c *= 2)
    if (std::fabs(std::log2(c / target)) < std::fabs(std::log2(best / target))) best = c;
  return best;
}

// Launch configuration of k_spgemm_rows for one product.
struct SpConfig {
  int lpr, W, H, rpb, threads;
  size_t lds;
};

static size_t spgemm_lds(int mode, int rpb, int W, int H, int per_row) {
  const size_t r = (size_t)rpb, h = (size_t)H;
  if (mode == SP_COUNT || mode == SP_BITS) return r * h * 4 + r * 4;
  if (mode == SP_FILL) return r * W * h * 8 + 2 * r * h * 4 + r * 4;
  return r * W * h * 8 + r * h * 4 + r * (per_row / kWave + 1) * 4;
}

// Lanes per sub-group from the mean row length of B; sub-groups per row so
// that each walks about eight entries of A; rows per block to fill 256
// threads.  W is halved until the block's LDS fits.
static SpConfig spgemm_config(ppe_solver* s, const Csr& A, const Csr& B, int mode, int H) {
  SpConfig c{};
  c.lpr = lanes_for(B);
  const double mean_a = A.n ? (double)A.nnz / A.n : 1.0;
  c.W = 1;
  while (c.W * c.lpr < 1024 && c.W < 16 && c.W * 8 < mean_a) c.W *= 2;
  c.H = H;
  while (true) {
    const int per_row = c.lpr * c.W;
    c.rpb = per_row >= kBlock ? 1 : kBlock / per_row;
    c.threads = c.rpb * per_row;
    c.lds = spgemm_lds(mode, c.rpb, c.W, H, per_row);
    if (c.lds <= s->lds_max || (c.W == 1 && c.rpb == 1)) break;
    if (c.W > 1) c.W /= 2;
    else c.lpr *= 2;  // fewer rows per block
  }
  require(c.lds <= s->lds_max, PPE_ERR_INTERNAL, "sparse product row does not fit in LDS");
  return c;
}

template <int MODE>
static void spgemm_launch(ppe_solver* s, const SpConfig& c, const Csr& A, const Csr& B,
                          const int* off, int stride, int* counts, int* cci, double* cv,
                          int* flag) {
  const int g = (A.n + c.rpb - 1) / c.rpb;
  const bool numeric = MODE == SP_FILL || MODE == SP_DENSE;
  const double* av = numeric ? A.v() : nullptr;
  const double* bv = numeric ? B.v() : nullptr;
#define PPE_SPR(L_)                                                                            \
  hipLaunchKernelGGL((k_spgemm_rows<L_, MODE>), dim3(g), dim3(c.threads), c.lds, s->stream, A.n, \
                     c.W, c.H, A.rp(), A.ci(), av, B.rp(), B.ci(), bv, off, stride, counts, cci,   \
                     cv, flag)
  switch (c.lpr) {
    case 4: PPE_SPR(4); break;
    case 8: PPE_SPR(8); break;
    case 16: PPE_SPR(16); break;
    case 32: PPE_SPR(32); break;
    default: PPE_SPR(64); break;
  }
#undef PPE_SPR
  PPE_LAUNCH_CHECK();
}

// C = A B.  Narrow products (C at most kSpDenseWidth columns, rows expected
// to fill a quarter of them) take one pass with a slot per column into
// fixed-stride scratch rows and a compaction; wider ones one pass of
// k_spgemm_wave into such rows, unless a row turns out longer than they are.
// Then, and where that is likely, or the scratch would be large or cannot be
// had, two passes count each row's distinct columns with a hash sized from the
// product bound (or a bit per column of C when that is smaller), then fill
// C with a hash sized from the largest count.  The
// product bound is maxrow(A) maxrow(B) when both are known on the host, else
// a bound pass reads it back.  C.maxrow is set to C's longest row.  extra: a
// device int read back in the same round trip as C's size (extra_host).
void spgemm(ppe_solver* s, const Csr& A, const Csr& B, Csr& C, int* flag, const int* extra,
            int* extra_host) {
  require(A.m == B.n, PPE_ERR_INTERNAL, "spgemm shape mismatch");
  C.n = A.n;
  C.m = B.m;
  int* crp = C.rowptr.get<int>(C.n + 1);
  if (C.n == 0) {
    C.nnz = 0;
    fill_int(s, crp, 0, 1);
    return;
  }
  int* counts = s->sp_cnt.get<int>(C.n + 1);
  int fm[2] = {0, 0};
  // flag[1] starts at 0 (zeroed below): counts are >= 0, so the max needs
  // no fill of its own unless a bound pass used the slot before
  bool max_slot_used = false;
  auto fetch_scan = [&](bool with_max, bool over = false) {
    // a bound pass that used the max slot leaves a larger value there
    if (with_max && max_slot_used) fill_int(s, flag + 1, INT32_MIN, 1);
    int none = 0;
    const long long total = exclusive_scan_read(
        s, counts, crp, C.n, with_max ? flag + 1 : nullptr,
        {ReadItem{flag, sizeof(int) * 2, fm},
         extra ? ReadItem{extra, sizeof(int), extra_host} : ReadItem{flag, sizeof(int), &none}});
    if (over && fm[0] != 0) return false;
    require(fm[0] == 0, PPE_ERR_INTERNAL, "sparse product row overflowed its hash table");
    require(total <= INT32_MAX, PPE_ERR_INTERNAL, "sparse product too large for int32 indices");
    C.nnz = total;
    C.maxrow = fm[1];
    return true;
  };

  const double mean_a = (double)A.nnz / A.n, mean_b = B.n ? (double)B.nnz / B.n : 0.0;
  if (C.m <= kSpDenseWidth && 4.0 * mean_a * mean_b >= C.m) {
    int H = 64;
    while (H < C.m) H += 64;
    const SpConfig c = spgemm_config(s, A, B, SP_DENSE, H);
    const size_t cap = (size_t)C.n * C.m;
    require(cap <= INT32_MAX, PPE_ERR_INTERNAL, "sparse product scratch too large");
    int* sci = s->sp_ci.get<int>(cap);
    double* sv = s->sp_v.get<double>(cap);
    spgemm_launch<SP_DENSE>(s, c, A, B, nullptr, C.m, counts, sci, sv, flag);
    fetch_scan(true);
    int* cci = C.col.get<int>(C.nnz);
    double* cv = C.val.get<double>(C.nnz);
    PPE_ROWS(lanes_for(B), k_spgemm_compact, C.n, C.n, C.m, crp, sci, sv, cci, cv);
    return;
  }

  int ub = C.m;  // the product bound, where both longest rows are known
  if (A.maxrow > 0 && B.maxrow > 0) ub = (int)std::min<int64_t>((int64_t)A.maxrow * B.maxrow, C.m);
  const bool few = C.n <= kSpFewRows;
  int wcap = 16;
  while (wcap < ub && wcap < (few ? kSpCapFew : kSpCap)) wcap *= 2;
  const int64_t cap = (int64_t)C.n * wcap;
  const bool fits = (int64_t)std::min<int64_t>(ub, (int64_t)kSpUnion * B.maxrow) <= wcap;
  int* sci = fits && cap <= kSpScratch ? s->sp_ci.try_get<int>(cap) : nullptr;
  double* sv = sci ? s->sp_v.try_get<double>(cap) : nullptr;
  if (sci && !sv) s->sp_ci.release();
  if (sv) {
    int hshift = 32;
    for (int h = 2 * wcap; h > 1; h /= 2) --hshift;
    const int lpr = lanes_for(B), W = mean_a * lpr > kSpSplit ? kSpWaves : 1, per = kSpWaves / W;
    const int g = (C.n + per - 1) / per;
#define PPE_SPW(L_, W_)                                                                          \
  hipLaunchKernelGGL((k_spgemm_wave<L_, W_>), dim3(g), dim3(kSpWaves * kWave),                   \
                     per * spgemm_wave_lds(wcap, W), s->stream, C.n, wcap, hshift, A.rp(),       \
                     A.ci(), A.v(), B.rp(), B.ci(), B.v(), counts, sci, sv, flag)
#define PPE_SPW_W(L_)             \
  if (W == 1) PPE_SPW(L_, 1);     \
  else PPE_SPW(L_, kSpWaves)
    switch (lpr) {
      case 4: PPE_SPW_W(4); break;
      case 8: PPE_SPW_W(8); break;
      case 16: PPE_SPW_W(16); break;
      case 32: PPE_SPW_W(32); break;
      default: PPE_SPW_W(64); break;
    }
#undef PPE_SPW_W
#undef PPE_SPW
    PPE_LAUNCH_CHECK();
    if (fetch_scan(true, true)) {
      int* cci = C.col.get<int>(C.nnz);
      double* cv = C.val.get<double>(C.nnz);
      PPE_ROWS(lanes_for(C), k_spgemm_compact, C.n, C.n, wcap, crp, sci, sv, cci, cv);
      return;
    }
    fill_int(s, flag, 0, 2);
  }

  if (A.maxrow <= 0 || B.maxrow <= 0) {
    int* prod = s->sp_prod.get<int>(C.n + 1);
    PPE_ROWS(lanes_for(A), k_spgemm_bound, C.n, C.n, A.rp(), A.ci(), B.rp(), prod);
    max_int_async(s, prod, C.n, flag + 1, false);
    max_slot_used = true;
    read_back(s, {ReadItem{flag, sizeof(int) * 2, fm}});
    ub = std::min(fm[1], C.m);
  }
  int Hc = 32;
  while (Hc < 2 * ub && Hc < 8192) Hc *= 2;
  // count with a bit per column of C when that takes less LDS than the hash
  const int words = (C.m + 31) / 32;
  if (words < Hc) {
    const SpConfig cb = spgemm_config(s, A, B, SP_BITS, words);
    spgemm_launch<SP_BITS>(s, cb, A, B, nullptr, 0, counts, nullptr, nullptr, flag);
  } else {
    const SpConfig cc = spgemm_config(s, A, B, SP_COUNT, Hc);
    spgemm_launch<SP_COUNT>(s, cc, A, B, nullptr, 0, counts, nullptr, nullptr, flag);
  }
  fetch_scan(true);
  int H = 16;  // at least twice the longest row: list and ckey hold H / 2
  while (H < 2 * fm[1]) H *= 2;
  const SpConfig cf = spgemm_config(s, A, B, SP_FILL, H);
  int* cci = C.col.get<int>(C.nnz);
  double* cv = C.val.get<double>(C.nnz);
  spgemm_launch<SP_FILL>(s, cf, A, B, crp, 0, nullptr, cci, cv, flag);
}

// T = A^T with sorted rows; returns where T's longest row is left (a device
// int, until the next transpose).
const int* transpose(ppe_solver* s, const Csr& A, Csr& T) {
  T.n = A.m;
  T.m = A.n;
  T.nnz = A.nnz;
  T.maxrow = 0;
  if (narrow_pays(T.n, A.nnz)) {
    int* trp = T.rowptr.get<int>(T.n + 1);
    hipLaunchKernelGGL(k_narrow_count, dim3(1), dim3(1024), 0, s->stream, A.nnz, T.n, A.ci(), trp,
                       s->cols.get<int>(1));
    PPE_LAUNCH_CHECK();
    int* rowid = s->tmp_i[2].get<int>(A.nnz);
    hipLaunchKernelGGL(k_row_ids, dim3(grid_for(A.n)), dim3(kBlock), 0, s->stream, A.n, A.rp(),
                       rowid);
    PPE_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_narrow_fill, dim3(T.n), dim3(1024), 0, s->stream, A.nnz, A.ci(), A.v(),
                       rowid, trp, T.col.get<int>(T.nnz), T.val.get<double>(T.nnz));
    PPE_LAUNCH_CHECK();
    return s->cols.as<int>();
  }
  // the counts and, behind them, the longest row
  int* cnt = s->cols.get<int>(T.n + 1);
  int* rmax = cnt + T.n;
  fill_int(s, cnt, 0, T.n + 1);
  int* pos = s->tmp_i[1].get<int>(A.nnz + 1);
  if (A.nnz) {
    hipLaunchKernelGGL(k_col_slots, dim3(grid_for(A.nnz, kSlotChunk)), dim3(kBlock), 0, s->stream,
                       A.nnz, A.ci(), cnt, pos);
    PPE_LAUNCH_CHECK();
  }
  int* trp = T.rowptr.get<int>(T.n + 1);
  exclusive_scan_async(s, cnt, trp, T.n, 0, rmax);  // the total is A.nnz
  int* tci = T.col.get<int>(T.nnz);
  double* tv = T.val.get<double>(T.nnz);
  int* uci = s->tmp_i[2].get<int>(T.nnz);
  double* uv = s->tmp_d[1].get<double>(T.nnz);
  if (A.n) {
    PPE_ROWS(lanes_for(A), k_transpose_fill, A.n, A.n, A.rp(), A.ci(), A.v(), trp, pos, uci, uv);
  }
  if (T.n) {
    hipLaunchKernelGGL(k_rank_rows, dim3(T.n), dim3(kWave), 0, s->stream, trp, uci, uv, tci, tv);
    PPE_LAUNCH_CHECK();
  }
  return rmax;
}

// The level's spectral bound of D^-1 A into *rho_dev (read back with the
// rest of the setup results): Gershgorin on the finest level, the safety
// factor times a power estimate on coarse ones.
void spectral_bound(ppe_solver* s, Level& L, int lvl, double* rho_dev) {
  const int n = L.n;
  if (n == 0) {
    fill_double(s, rho_dev, 1.0, 1);
    return;
  }
  if (lvl == 0) {
    const int g = grid_for(n);
    double* part = s->tmp_d[0].get<double>(g);
#define PPE_GERSH(WM_)                                                                        \
  hipLaunchKernelGGL(k_gershgorin_ell<WM_>, dim3(g), dim3(kBlock), 0, s->stream, n, L.W,       \
                     L.ell_col.as<int>(), L.ell_val.as<double>(), L.diag.as<double>(), part)
    if (L.W <= 0 || L.W > 8)
      hipLaunchKernelGGL(k_gershgorin, dim3(g), dim3(kBlock), 0, s->stream, n, L.A.rp(), L.A.v(),
                         L.diag.as<double>(), part);
    else if (L.W <= 4) PPE_GERSH(4);
    else if (L.W <= 6) PPE_GERSH(6);
    else PPE_GERSH(8);
#undef PPE_GERSH
    PPE_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_max_partials, dim3(1), dim3(kBlock), 0, s->stream, part, g, rho_dev);
    PPE_LAUNCH_CHECK();
    return;
  }
  L.x.get<double>(n);
  L.r.get<double>(n);
  // setup work: its power steps stay out of the solve's kernel profile
  struct NoProfile {
    ppe_solver* s;
    bool saved;
    ~NoProfile() { s->prof = saved; }
  } guard{s, s->prof};
  s->prof = false;
  power_estimate(s, L, level_salt(lvl), kPowerIters, kPowerSafety, rho_dev);
}

// Launches inside the scope go to another stream of the solver.
struct OnStream {
  ppe_solver* s;
  hipStream_t saved;
  OnStream(ppe_solver* s_, hipStream_t st) : s(s_), saved(s_->stream) { s->stream = st; }
  ~OnStream() { s->stream = saved; }
};

void ensure_side_stream(ppe_solver* s) {
  if (s->side) return;
  PPE_HIP(hipStreamCreateWithFlags(&s->side, hipStreamNonBlocking));
  PPE_HIP(hipEventCreateWithFlags(&s->fork_ev, hipEventDisableTiming));
  PPE_HIP(hipEventCreateWithFlags(&s->join_ev, hipEventDisableTiming));
}

}  // namespace

// ---- coarse levels kept across a changed mask
namespace {

// Row i of the re-indexed finest prolongator: the base build's row of the
// same cell, or empty for a pin or a cell that build did not have.  cnt[i]
// is its length; matched[i] = 1 if the cell had a row in the base build.
__global__ void k_reuse_rows(int na, const int* __restrict__ perm, const int* __restrict__ comp,
                             const int* __restrict__ base_cid, const int* __restrict__ base_rp,
                             int* __restrict__ cnt, int* __restrict__ matched) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= na) return;
  const int c = perm[i];
  const int o = base_cid[c];
  cnt[i] = (o >= 0 && comp[c] != c) ? base_rp[o + 1] - base_rp[o] : 0;
  matched[i] = o >= 0 ? 1 : 0;
}

__global__ void k_reuse_fill(int na, const int* __restrict__ perm, const int* __restrict__ comp,
                             const int* __restrict__ base_cid, const int* __restrict__ base_rp,
                             const int* __restrict__ base_ci, const double* __restrict__ base_v,
                             const int* __restrict__ rp, int* __restrict__ ci,
                             double* __restrict__ v) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= na) return;
  const int c = perm[i];
  const int o = base_cid[c];
  if (o < 0 || comp[c] == c) return;
  const int src = base_rp[o], len = base_rp[o + 1] - src, dst = rp[i];
  for (int k = 0; k < len; ++k) {
    ci[dst + k] = base_ci[src + k];
    v[dst + k] = base_v[src + k];
  }
}

}  // namespace

void keep_base(ppe_solver* s) {
  s->have_base = false;
  if (s->opt.coarse_reuse <= 0 || s->shifted || s->nlev < 2) return;
  const int nc = s->n_cells;
  const Csr& P = s->levels[0].P;
  Csr& B = s->base_P0;
  B.n = P.n;
  B.m = P.m;
  B.nnz = P.nnz;
  B.maxrow = P.maxrow;
  PPE_HIP(hipMemcpyAsync(s->base_cid.get<int>(nc + 1), s->cid.as<int>(), sizeof(int) * (nc + 1),
                         hipMemcpyDeviceToDevice, s->stream));
  PPE_HIP(hipMemcpyAsync(B.rowptr.get<int>(P.n + 1), P.rp(), sizeof(int) * (P.n + 1),
                         hipMemcpyDeviceToDevice, s->stream));
  if (P.nnz) {
    PPE_HIP(hipMemcpyAsync(B.col.get<int>(P.nnz), P.ci(), sizeof(int) * P.nnz,
                           hipMemcpyDeviceToDevice, s->stream));
    PPE_HIP(hipMemcpyAsync(B.val.get<double>(P.nnz), P.v(), sizeof(double) * P.nnz,
                           hipMemcpyDeviceToDevice, s->stream));
  }
  s->base_na = s->n_active;
  s->base_nlev = s->nlev;
  s->base_uses = 0;
  s->have_base = true;
}

bool reuse_coarse_levels(ppe_solver* s) {
  if (!s->have_base || s->shifted || s->base_uses >= s->opt.coarse_reuse) return false;
  const int na = s->n_active;
  if (na == 0) return false;
  Level& L0 = s->levels[0];
  const Csr& B = s->base_P0;
  const int* perm = s->perm.as<int>();
  const int* comp = s->comp_full.as<int>();
  const int* bcid = s->base_cid.as<int>();
  int* cnt = s->tmp_i[0].get<int>(na + 1);
  int* matched = s->tmp_i[1].get<int>(na + 1);
  hipLaunchKernelGGL(k_reuse_rows, dim3(grid_for(na)), dim3(kBlock), 0, s->stream, na, perm, comp,
                     bcid, B.rp(), cnt, matched);
  PPE_LAUNCH_CHECK();
  int* rp = L0.P.rowptr.get<int>(na + 1);
  const long long* d_nnz = exclusive_scan_async(s, cnt, rp, na, 0);
  const long long* d_matched = exclusive_scan_async(s, matched, s->tmp_i[2].get<int>(na + 1), na, 1);
  const double* d_rho = level0_bound_async(s);
  long long nnz = 0, kept = 0;
  double rho = 0.0;
  read_back(s, {ReadItem{d_nnz, sizeof(long long), &nnz},
                ReadItem{d_matched, sizeof(long long), &kept},
                ReadItem{d_rho, sizeof(double), &rho}});
  // cells removed since the base build plus cells it did not have
  const long long moved = (s->base_na - kept) + (na - kept);
  if (10 * moved > (long long)s->base_na) return false;
  Csr& P = L0.P;
  P.n = na;
  P.m = B.m;
  P.nnz = nnz;
  P.maxrow = B.maxrow;
  hipLaunchKernelGGL(k_reuse_fill, dim3(grid_for(na)), dim3(kBlock), 0, s->stream, na, perm, comp,
                     bcid, B.rp(), B.ci(), B.v(), rp, P.col.get<int>(nnz > 0 ? nnz : 1),
                     P.val.get<double>(nnz > 0 ? nnz : 1));
  PPE_LAUNCH_CHECK();
  transpose(s, P, L0.R);
  L0.n_agg = B.m;
  L0.rho = rho;
  L0.ap_ok = false;
  L0.dense = false;
  s->nlev = s->base_nlev;
  s->base_uses += 1;
  return true;
}

const double* level0_bound_async(ppe_solver* s) {
  double* out = s->setup_out.get<double>((size_t)std::max(1, s->opt.max_levels) + 1);
  spectral_bound(s, s->levels[0], 0, out);
  return out;
}

// P on the finest level from its ELL copy (k_coarsen_cols_ell): count, scan
// with the longest row (one round trip), fill.  P is what the general product
// and k_smooth_p give, entry for entry.
static void coarsen_cols_ell(ppe_solver* s, const Level& L, const int* agg, const double* pt,
                             int na, const double* rho, Csr& P, int* flag) {
  const int n = L.n, W = L.W;
  P.n = n;
  P.m = na;
  int* prp = P.rowptr.get<int>(n + 1);
  int* counts = s->sp_cnt.get<int>(n + 1);
  const int g = grid_for(n);
  const int* ecol = L.ell_col.as<int>();
  const double* ev = L.ell_val.as<double>();
  const double* dg = L.diag.as<double>();
#define PPE_QC(WM, COUNT, ...)                                                                 \
  hipLaunchKernelGGL((k_coarsen_cols_ell<WM, COUNT>), dim3(g), dim3(kBlock), 0, s->stream, n, W, \
                     ecol, ev, dg, agg, pt, rho, __VA_ARGS__)
  if (W <= 4) PPE_QC(4, true, counts, nullptr, nullptr, nullptr);
  else if (W <= 6) PPE_QC(6, true, counts, nullptr, nullptr, nullptr);
  else PPE_QC(8, true, counts, nullptr, nullptr, nullptr);
  PPE_LAUNCH_CHECK();
  int fm[2] = {0, 0};
  const long long total = exclusive_scan_read(s, counts, prp, n, flag + 1,
                                              {ReadItem{flag, sizeof(int) * 2, fm}});
  require(total <= INT32_MAX, PPE_ERR_INTERNAL, "sparse product too large for int32 indices");
  P.nnz = total;
  P.maxrow = fm[1];
  int* pci = P.col.get<int>(P.nnz + kApU);
  double* pv = P.val.get<double>(P.nnz + kApU);
  if (W <= 4) PPE_QC(4, false, nullptr, prp, pci, pv);
  else if (W <= 6) PPE_QC(6, false, nullptr, prp, pci, pv);
  else PPE_QC(8, false, nullptr, prp, pci, pv);
#undef PPE_QC
  PPE_LAUNCH_CHECK();
}

// AP = A P on the finest level from its ELL copy (k_ap_merge_ell): count,
// scan with the longest row and the device value extra (one round trip),
// fill.
static void ap_merge_ell(ppe_solver* s, const Level& L, const Csr& P, Csr& AP, int* flag,
                         const int* extra, int* extra_host) {
  const int n = L.n, W = L.W;
  AP.n = n;
  AP.m = P.m;
  int* crp = AP.rowptr.get<int>(n + 1);
  int* counts = s->sp_cnt.get<int>(n + 1);
  const int g = grid_for(n);
  const int* ecol = L.ell_col.as<int>();
  const double* ev = L.ell_val.as<double>();
  const double* dg = L.diag.as<double>();
#define PPE_AP(WM, COUNT, ...)                                                                 \
  hipLaunchKernelGGL((k_ap_merge_ell<WM, COUNT>), dim3(g), dim3(kBlock), 0, s->stream, n, W, ecol, \
                     ev, dg, P.rp(), P.ci(), P.v(), __VA_ARGS__)
  if (W <= 4) PPE_AP(4, true, counts, nullptr, nullptr, nullptr);
  else if (W <= 6) PPE_AP(6, true, counts, nullptr, nullptr, nullptr);
  else PPE_AP(8, true, counts, nullptr, nullptr, nullptr);
  PPE_LAUNCH_CHECK();
  int fm[2] = {0, 0};
  const long long total = exclusive_scan_read(
      s, counts, crp, n, flag + 1,
      {ReadItem{flag, sizeof(int) * 2, fm}, ReadItem{extra, sizeof(int), extra_host}});
  require(total <= INT32_MAX, PPE_ERR_INTERNAL, "sparse product too large for int32 indices");
  AP.nnz = total;
  AP.maxrow = fm[1];
  int* cci = AP.col.get<int>(AP.nnz);
  double* cv = AP.val.get<double>(AP.nnz);
  if (W <= 4) PPE_AP(4, false, nullptr, crp, cci, cv);
  else if (W <= 6) PPE_AP(6, false, nullptr, crp, cci, cv);
  else PPE_AP(8, false, nullptr, crp, cci, cv);
#undef PPE_AP
  PPE_LAUNCH_CHECK();
}

void build_hierarchy(ppe_solver* s) {
  const int maxlev = std::max(1, s->opt.max_levels);
  // spectral bounds, the error word, then each level's three products' error
  // bits and longest rows, all cleared at once
  double* rho_dev = s->setup_out.get<double>((size_t)maxlev + 1 + 3 * maxlev);
  int* err = reinterpret_cast<int*>(rho_dev + maxlev);
  fill_int(s, reinterpret_cast<int*>(rho_dev), 0, 2 * ((int64_t)maxlev + 1 + 3 * maxlev));
  for (int lvl = 0;; ++lvl) {
    Level& L = s->levels[lvl];
    const int n = L.n;
    // setup kernels use the fixed launch rules: choices the autotuner made
    // for the previous hierarchy would change the order of the power
    // iteration's sums, and with it the spectral bound
    L.lpr_a = L.lpr_r = L.lpr_p = 0;
    L.fuse0 = true;
    L.ap_ok = false;
    L.op_ok = false;
    if (lvl > 0 && n > 0) {
      PPE_ROWS(lanes_for(L.A), k_diag, n, n, L.A.rp(), L.A.ci(), L.A.v(), L.diag.get<double>(n),
               err);  // sets SE_DIAG
    }
    L.n_agg = 0;
    L.dense = false;
    const bool last = n <= s->opt.coarse_max || lvl == s->opt.max_levels - 1;
    // a coarsest level solved by its explicit inverse runs no smoother and
    // has no prolongator to smooth: its spectral bound is never used.  A
    // coarse level's power estimate (a chain of small launches) runs on the
    // side stream beside the strength, MIS-2 and aggregation launches,
    // which do not need it; the prolongator smoothing waits for it.
    bool joined = true;
    auto join = [&]() {
      if (!joined) {
        PPE_HIP(hipStreamWaitEvent(s->stream, s->join_ev, 0));
        joined = true;
      }
    };
    if (last && n > 0 && n <= kDenseMax) {
      // rho stays 0
    } else if (lvl > 0 && n > 0) {
      ensure_side_stream(s);
      PPE_HIP(hipEventRecord(s->fork_ev, s->stream));
      PPE_HIP(hipStreamWaitEvent(s->side, s->fork_ev, 0));
      {
        OnStream on(s, s->side);
        spectral_bound(s, L, lvl, rho_dev + lvl);
      }
      PPE_HIP(hipEventRecord(s->join_ev, s->side));
      joined = false;
    } else {
      spectral_bound(s, L, lvl, rho_dev + lvl);
    }
    if (!last) {
      const int g = grid_for(n);
      // the finest level runs these passes on its ELL copy (one thread per
      // row); coarse levels on CSR with lpr lanes per row
      const bool ell = lvl == 0 && L.W > 0;
      const int W = L.W;
      const int* ecol = L.ell_col.as<int>();
      const double* ev = L.ell_val.as<double>();
      unsigned char* strong = ell ? nullptr : L.strong.get<unsigned char>(L.A.nnz);
      int* scol = ell ? L.scol.get<int>((size_t)W * n) : nullptr;
      unsigned char* st = L.state.get<unsigned char>(n);
      unsigned long long* m1 = L.m1.get<unsigned long long>(n);
      const int lpr = agg_lanes(L.A);
#define PPE_SLOTS(LAUNCH)                      \
  do {                                         \
    if (W <= 4) { LAUNCH(4); }                 \
    else if (W <= 6) { LAUNCH(6); }            \
    else if (W <= 8) { LAUNCH(8); }            \
    else { LAUNCH(0); }                        \
    PPE_LAUNCH_CHECK();                        \
  } while (0)
#define PPE_ELL_K(K, ...) \
  hipLaunchKernelGGL(K, dim3(g), dim3(kBlock), 0, s->stream, __VA_ARGS__)
      // the threshold is halved (theta_decay) on each coarser level
      const double theta_l = s->opt.theta * std::pow(s->opt.theta_decay, lvl);
      if (ell) {
#define PPE_L(WM) PPE_ELL_K(k_strength_ell<WM>, n, W, ecol, ev, L.diag.as<double>(), theta_l * theta_l, scol, st)
        PPE_SLOTS(PPE_L);
#undef PPE_L
      } else {
        PPE_ROWS(lpr, k_strength, n, n, L.A.rp(), L.A.ci(), L.A.v(), L.diag.as<double>(),
                 theta_l * theta_l, strong, st);
      }
      const uint32_t salt = level_salt(lvl);
      // As many rounds before the first host check as any set-up of this level has
      // launched so far (mis_batch never falls), then a few at a time (on the finest
      // level the later ones are k_mis_finish_ell's); a round after the set is
      // complete changes nothing.
      // The roots are numbered before each check and their count read with it:
      // the numbering is kept once no node is left undecided.
      int* und = s->tmp_i[3].get<int>(1);
      int* root = s->tmp_i[2].get<int>(n + 1);
      int* root_id = L.mis_root.get<int>(n + 1);
      long long n_roots = 0;
      const int64_t entries = ell ? (int64_t)W * n : L.A.nnz;
      const size_t lds = mis_small_lds(n, entries, !ell);
      if (n <= 0xFFFF && entries <= kMisEntries && lds + kMisStatic <= s->lds_max) {
        int l1 = 1;  // lanes per row: no more than fill the workgroup
        while (l1 < 16 && 2 * l1 * n <= kMisThreads) l1 *= 2;
        long long* total = s->tmp_l[0].get<long long>(2);
        hipLaunchKernelGGL(k_mis_small, dim3(1), dim3(kMisThreads), lds, s->stream, n, l1, W, scol,
                           ell ? nullptr : L.A.rp(), L.A.ci(), strong, salt, st, root_id, total);
        PPE_LAUNCH_CHECK();
        read_back(s, {ReadItem{total, sizeof(long long), &n_roots}});
      } else {
        int rounds = 0;
        for (int batch = std::max(ell ? kMisRounds + 4 : 3, L.mis_batch);; batch = ell ? 2 : 3) {
          for (int k = 0; k < batch; ++k, ++rounds) {
            if (k == batch - 1) fill_int(s, und, 0, 1);
            if (!ell) {
              PPE_ROWS(lpr, k_mis_max1, n, n, L.A.rp(), L.A.ci(), strong, st, salt, m1);
              PPE_ROWS(lpr, k_mis_max2, n, n, L.A.rp(), L.A.ci(), strong, st, salt, m1, und);
            } else if (rounds < kMisRounds) {
#define PPE_L(WM) PPE_ELL_K(k_mis_max1_ell<WM>, n, W, scol, st, salt, m1)
              PPE_SLOTS(PPE_L);
#undef PPE_L
#define PPE_L(WM) PPE_ELL_K(k_mis_max2_ell<WM>, n, W, scol, st, salt, m1)
              PPE_SLOTS(PPE_L);
#undef PPE_L
            } else {
#define PPE_L(WM)                                                                           \
  hipLaunchKernelGGL(k_mis_finish_ell<WM>, dim3(grid_for(n, kFinishRows)), dim3(kBlock), 0, \
                     s->stream, n, W, scol, st, salt, und)
              PPE_SLOTS(PPE_L);
#undef PPE_L
            }
          }
          hipLaunchKernelGGL(k_is_root, dim3(g), dim3(kBlock), 0, s->stream, n, st, root);
          PPE_LAUNCH_CHECK();
          int left = 0;
          n_roots = exclusive_scan_read(s, root, root_id, n, nullptr,
                                        {ReadItem{und, sizeof(int), &left}});
          if (left == 0) break;
          require(rounds < 10000, PPE_ERR_INTERNAL, "MIS-2 did not terminate");
        }
        L.mis_batch = rounds;
      }
      const int na = (int)n_roots;
      if (na > 0) {
        int* agg1 = L.agg1.get<int>(n);
        int* agg = L.agg.get<int>(n);
        if (ell) {
#define PPE_L(WM) PPE_ELL_K(k_agg_first_ell<WM>, n, W, scol, st, root_id, agg1)
          PPE_SLOTS(PPE_L);
#undef PPE_L
#define PPE_L(WM) PPE_ELL_K(k_agg_second_ell<WM>, n, W, scol, ev, agg1, agg, err)
          PPE_SLOTS(PPE_L);  // sets SE_AGG
#undef PPE_L
        } else {
          PPE_ROWS(lpr, k_agg_first, n, n, L.A.rp(), L.A.ci(), strong, st, root_id, agg1);
          PPE_ROWS(lpr, k_agg_second, n, n, L.A.rp(), L.A.ci(), L.A.v(), strong, agg1, agg,
                   err);  // sets SE_AGG
        }
#undef PPE_ELL_K
#undef PPE_SLOTS
        L.n_agg = na;
        // aggregate members, coarse near-null vector, tentative prolongator
        // (nodes with no strong connection stay outside every aggregate, so
        // members and prolongator entries number at most n; only the device
        // row pointers are exact)
        int* cnt = s->tmp_i[0].get<int>(na + 1);
        fill_int(s, cnt, 0, na + 1);
        int* pos = s->tmp_i[1].get<int>(n);
        hipLaunchKernelGGL(k_col_slots, dim3(grid_for(n, kSlotChunk)), dim3(kBlock), 0, s->stream,
                           (int64_t)n, agg, cnt, pos);
        PPE_LAUNCH_CHECK();
        int* aptr = L.agg_ptr.get<int>(na + 1);
        exclusive_scan_async(s, cnt, aptr, na);
        int* mem = L.agg_mem.get<int>(n);
        hipLaunchKernelGGL(k_agg_fill, dim3(g), dim3(kBlock), 0, s->stream, n, agg, aptr, pos, mem);
        PPE_LAUNCH_CHECK();
        if ((int)s->levels.size() < lvl + 2) s->levels.resize(lvl + 2);
        Level& L0 = s->levels[lvl];  // re-fetch: resize may move levels
        Level& C = s->levels[lvl + 1];
        double* Bc = C.B.get<double>(na);
        hipLaunchKernelGGL(k_agg_norm, dim3(grid_for((int64_t)na * kWave / 2 + kWave)), dim3(kBlock), 0,
                           s->stream, na, aptr, mem, L0.B.as<double>(), Bc);
        PPE_LAUNCH_CHECK();
        double* pt = L0.pt.get<double>(n);
        int* pcnt = s->tmp_i[0].get<int>(n + 1);
        hipLaunchKernelGGL(k_tent, dim3(g), dim3(kBlock), 0, s->stream, n, agg, L0.B.as<double>(), Bc,
                           pcnt, pt);
        PPE_LAUNCH_CHECK();
        int* flag = reinterpret_cast<int*>(rho_dev + maxlev + 1 + 3 * lvl);
        const bool merge = lvl == 0 && L0.W > 0 && L0.W <= 8;
        // smoothed prolongator (with this level's spectral bound)
        Csr& P = L0.P;
        P.n = n;
        P.m = na;
        if (merge) {
          join();
          coarsen_cols_ell(s, L0, agg, pt, na, rho_dev + lvl, P, flag);
        } else {
          Csr& Pt = L0.Pt;
          Pt.n = n;
          Pt.m = na;
          Pt.maxrow = 1;
          int* ptrp = Pt.rowptr.get<int>(n + 1);
          exclusive_scan_async(s, pcnt, ptrp, n);
          Pt.nnz = n;  // capacity (an upper bound): only the row pointers are read
          hipLaunchKernelGGL(k_tent_csr, dim3(g), dim3(kBlock), 0, s->stream, n, ptrp, agg, pt,
                             Pt.col.get<int>(Pt.nnz), Pt.val.get<double>(Pt.nnz));
          PPE_LAUNCH_CHECK();
          spgemm(s, L0.A, Pt, L0.Q, flag, nullptr, nullptr);
          P.nnz = L0.Q.nnz;
          P.maxrow = L0.Q.maxrow;
          join();
          hipLaunchKernelGGL(k_smooth_p, dim3(g), dim3(kBlock), 0, s->stream, n, L0.Q.rp(),
                             L0.Q.ci(), L0.Q.v(), L0.diag.as<double>(), agg, pt, rho_dev + lvl,
                             P.val.get<double>(P.nnz));
          PPE_LAUNCH_CHECK();
          // P has the pattern of A P_tent: take its arrays instead of copying
          std::swap(P.rowptr, L0.Q.rowptr);
          std::swap(P.col, L0.Q.col);
        }
        const int* rmax = transpose(s, P, L0.R);
        if (merge)
          ap_merge_ell(s, L0, P, L0.AP, flag + 2, rmax, &L0.R.maxrow);
        else
          spgemm(s, L0.A, P, L0.AP, flag + 2, rmax, &L0.R.maxrow);
        L0.ap_ok = true;
        spgemm(s, L0.R, L0.AP, C.A, flag + 4, nullptr, nullptr);
        C.n = na;
        s->nlev = lvl + 2;
        continue;
      }
    }
    // coarsest level
    join();
    s->nlev = lvl + 1;
    if (n > 0 && n <= kDenseMax) {
      // the blocked form's matrix is padded to whole blocks
      const int nb = (n + kGinvB - 1) / kGinvB, N = n <= kDenseBlk ? n : kGinvB * nb;
      double* Ainv = L.Ainv.get<double>((size_t)N * N);
      L.inv_ld = N;
      double* G0 = s->tmp_d[1].get<double>((size_t)N * N + 2 * kGinvB * kGinvB);
      double* Dinv = G0 + (size_t)N * N;
      double* Dnext = Dinv + kGinvB * kGinvB;
      double* G1 = Ainv;
      // the last of the block steps, which alternate between the two, writes Ainv
      if (n > kDenseBlk && nb % 2 == 0) std::swap(G0, G1);
      hipLaunchKernelGGL(k_densify, dim3(N), dim3(kBlock), 0, s->stream, n, N, L.A.rp(), L.A.ci(),
                         L.A.v(), G0);
      PPE_LAUNCH_CHECK();
      if (n <= kDenseBlk) {
        hipLaunchKernelGGL(k_dense_inverse_blk, dim3(1), dim3(1024), 0, s->stream, n, G0, Ainv, err);
      } else {
        hipLaunchKernelGGL(k_ginv_first, dim3(1), dim3(256), 0, s->stream, N, G0, Dinv, err);
        for (int K = 0; K < nb; ++K) {
          PPE_LAUNCH_CHECK();
          hipLaunchKernelGGL(k_ginv_step, dim3(nb, nb), dim3(256), 0, s->stream, N, G0, Dinv, K, G1,
                             Dnext, err);
          std::swap(G0, G1);
          std::swap(Dinv, Dnext);
        }
      }
      PPE_LAUNCH_CHECK();
      L.dense = true;
    }
    break;
  }
  // one read-back for the whole hierarchy: spectral bounds and error bits
  std::vector<double> out((size_t)maxlev + 1);
  read_back(s, {ReadItem{rho_dev, sizeof(double) * (maxlev + 1), out.data()}});
  int bits = 0;
  std::memcpy(&bits, &out[maxlev], sizeof(int));
  require(!(bits & SE_DIAG), PPE_ERR_INTERNAL, "coarse operator lost its diagonal");
  require(!(bits & SE_AGG), PPE_ERR_INTERNAL, "aggregation left a node unassigned");
  require(!(bits & SE_DENSE), PPE_ERR_INTERNAL, "coarsest operator is not positive definite");
  for (int l = 0; l < s->nlev; ++l) s->levels[l].rho = out[l];
}

}  // namespace ppe
