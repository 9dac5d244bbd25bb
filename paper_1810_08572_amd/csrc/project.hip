// Pressure-correction step with the cross-diffusion term of the face-gradient
// split (section 2.3, Eq. 11-12), the solidification changes to the face
// gradient (section 2.4.2, cases 2 and 3, Eq. 15-16), and the consistent face
// volume flux and velocity correction (section 2.4.3, Eq. 17 and Eq. 8).
//
// Face gradient: at an interior face with owner C1, neighbour C2 and
// vertices V1..V4, J has rows C2-C1, V3-V1, V4-V2 and
//   grad(phi)_f = J^-1 [phi_C2 - phi_C1, phi_V3 - phi_V1, phi_V4 - phi_V2],
// each vertex value the mean over the cells sharing that vertex.  This is a
// stencil over the face's neighbour cells (every cell sharing one of its
// vertices).  Case 2 (a solid neighbour cell) removes the solid cells and
// spreads their summed coefficients equally over the remaining ones, which
// is the same as giving every solid cell the mean value m_f of the face's
// remaining neighbour cells.  So only J^-1 is stored per face; each pass
// forms, per vertex, pbar_V = (sum of p over its active cells) / n_V and
// w_V = (its solid cells) / n_V, and a face uses pbar_V + w_V m_f, with m_f
// found by a merge of its vertices' sorted cell lists only where some w_V is
// not zero (the faces next to the front).
//
// The pressure equation with both terms, for active cell i:
//   (L p)_i - (X p)_i = b_i,
//   (L p)_i = sum_{open f} c_f (p_i - p_nb),
//   (X p)_i = sum_{open f} s_if t_f . grad(p)_f,   t_f = S_f/rho - c_f d_f,
//   b_i     = -(1/dt) sum_{open f} s_if F*_f,      F*_f = u*_f . S_f,
// (s_if = +1 when i owns f) is solved by deferred correction around the
// symmetric direct system that ppe_assemble set up: r = b + X p - L p on the
// non-pinned active cells, A delta = r by AMG-PCG, p += delta, until
// ||r|| <= rtol ||b||.  X is a small perturbation of L on meshes of moderate
// skewness, so each pass gains a fixed factor.
#include "common.h"

#include <algorithm>
#include <cmath>

namespace ppe {
namespace {

constexpr int kMaxValence = 16;  // cells per vertex
enum GeomErr { GE_INDEX = 1, GE_VALENCE = 2, GE_CORNER = 4, GE_SINGULAR = 8, GE_REPEAT = 16 };

__global__ void k_vertex_count(int n_cells, int n_nodes, const int* __restrict__ cell_nodes,
                               int* __restrict__ cnt, int* __restrict__ flag) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= n_cells) return;
  int v[8];
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    v[k] = cell_nodes[8 * (size_t)c + k];
    ok = ok && v[k] >= 0 && v[k] < n_nodes;
  }
  if (!ok) {
    atomicOr(flag, GE_INDEX);
    return;
  }
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = a + 1; b < 8; ++b)
      if (v[a] == v[b]) ok = false;
  if (!ok) {
    atomicOr(flag, GE_REPEAT);
    return;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) atomicAdd(cnt + v[k], 1);
}

__global__ void k_vertex_fill(int n_cells, const int* __restrict__ cell_nodes,
                              int* __restrict__ cursor, int* __restrict__ vcell) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= n_cells) return;
#pragma unroll
  for (int k = 0; k < 8; ++k) vcell[atomicAdd(cursor + cell_nodes[8 * (size_t)c + k], 1)] = c;
}

// ascending cell ids per vertex (placement order above is arbitrary)
__global__ void k_vertex_sort(int n_nodes, const int* __restrict__ vptr, int* __restrict__ vcell,
                              int* __restrict__ flag) {
  const int v = blockIdx.x * kBlock + threadIdx.x;
  if (v >= n_nodes) return;
  const int a = vptr[v], n = vptr[v + 1] - a;
  if (n > kMaxValence) {
    atomicOr(flag, GE_VALENCE);
    return;
  }
  for (int i = 1; i < n; ++i) {
    const int x = vcell[a + i];
    int j = i - 1;
    while (j >= 0 && vcell[a + j] > x) {
      vcell[a + j + 1] = vcell[a + j];
      --j;
    }
    vcell[a + j + 1] = x;
  }
}

__device__ __forceinline__ void cross3(const double* a, const double* b, double* c) {
  c[0] = a[1] * b[2] - a[2] * b[1];
  c[1] = a[2] * b[0] - a[0] * b[2];
  c[2] = a[0] * b[1] - a[1] * b[0];
}

// Local frame of interior face f: the columns of J^-1, stored as nine arrays
// (gi[k * n_faces + f], k = 3 column + component), g0 = (r1 x r2)/det,
// g1 = (r2 x r0)/det, g2 = (r0 x r1)/det for the rows r0 = C2 - C1,
// r1 = V3 - V1, r2 = V4 - V2.  Checks that both cells have all four vertices
// as corners and that the frame is not degenerate.  Walls get zeros.
__global__ void k_face_frame(int n_faces, int n_nodes, const int* __restrict__ owner,
                             const int* __restrict__ neigh, const int* __restrict__ face_nodes,
                             const int* __restrict__ vptr, const int* __restrict__ vcell,
                             const double* __restrict__ X, const double* __restrict__ C,
                             double* __restrict__ gi, int* __restrict__ flag) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  const int o = owner[f], n = neigh[f];
  double g[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (n >= 0) {
    int vv[4];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      vv[k] = face_nodes[4 * (size_t)f + k];
      ok = ok && vv[k] >= 0 && vv[k] < n_nodes;
    }
    if (!ok) {
      atomicOr(flag, GE_INDEX);
    } else {
      bool corner = true;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        bool has_o = false, has_n = false;
        for (int e = vptr[vv[k]]; e < vptr[vv[k] + 1]; ++e) {
          has_o = has_o || vcell[e] == o;
          has_n = has_n || vcell[e] == n;
        }
        corner = corner && has_o && has_n;
      }
      if (!corner) atomicOr(flag, GE_CORNER);
      double r0[3], r1[3], r2[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        r0[d] = C[3 * (size_t)n + d] - C[3 * (size_t)o + d];
        r1[d] = X[3 * (size_t)vv[2] + d] - X[3 * (size_t)vv[0] + d];
        r2[d] = X[3 * (size_t)vv[3] + d] - X[3 * (size_t)vv[1] + d];
      }
      cross3(r1, r2, g);
      cross3(r2, r0, g + 3);
      cross3(r0, r1, g + 6);
      const double det = r0[0] * g[0] + r0[1] * g[1] + r0[2] * g[2];
      const double scale = sqrt((r0[0] * r0[0] + r0[1] * r0[1] + r0[2] * r0[2]) *
                                (r1[0] * r1[0] + r1[1] * r1[1] + r1[2] * r1[2]) *
                                (r2[0] * r2[0] + r2[1] * r2[1] + r2[2] * r2[2]));
      if (!(fabs(det) > 1e-12 * scale)) {
        atomicOr(flag, GE_SINGULAR);
#pragma unroll
        for (int k = 0; k < 9; ++k) g[k] = 0.0;
      } else {
        const double inv_det = 1.0 / det;
#pragma unroll
        for (int k = 0; k < 9; ++k) g[k] *= inv_det;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) gi[(size_t)k * n_faces + f] = g[k];
}

__device__ __forceinline__ bool open_face(const int* active, int o, int n) {
  return n >= 0 && active[o] && active[n];
}

// F*_f = mean of the owners' u* dotted with S_f on open faces, else 0
__global__ void k_star_flux(int n_faces, const int* __restrict__ owner,
                            const int* __restrict__ neigh, const int* __restrict__ active,
                            const double* __restrict__ u, const double* __restrict__ S,
                            double* __restrict__ Fs) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  const int o = owner[f], n = neigh[f];
  double F = 0.0;
  if (open_face(active, o, n)) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
      F += 0.5 * (u[3 * (size_t)o + d] + u[3 * (size_t)n + d]) * S[3 * (size_t)f + d];
  }
  Fs[f] = F;
}

// b_i = -(1/dt) sum_{open f} s_if F*_f on active cells, 0 elsewhere
__global__ void k_rhs_from_flux(int n_cells, const int* __restrict__ adj_ptr,
                                const int* __restrict__ adj_nbr, const int* __restrict__ adj_face,
                                const int* __restrict__ owner, const int* __restrict__ active,
                                const double* __restrict__ Fs, double inv_dt,
                                double* __restrict__ b) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= n_cells) return;
  double s = 0.0;
  if (active[c]) {
    for (int e = adj_ptr[c]; e < adj_ptr[c + 1]; ++e) {
      if (!active[adj_nbr[e]]) continue;
      const int f = adj_face[e];
      s += owner[f] == c ? Fs[f] : -Fs[f];
    }
  }
  b[c] = -inv_dt * s;
}

// t_f = S_f / rho - c_f (C2 - C1) on interior faces (three arrays of n_faces)
__global__ void k_cross_vectors(int n_faces, const int* __restrict__ owner,
                                const int* __restrict__ neigh, const double* __restrict__ S,
                                const double* __restrict__ C, const double* __restrict__ coeff,
                                double inv_rho, double* __restrict__ t) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  const int o = owner[f], n = neigh[f];
  const double cf = n >= 0 ? coeff[f] : 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    t[(size_t)d * n_faces + f] =
        n >= 0 ? S[3 * (size_t)f + d] * inv_rho - cf * (C[3 * (size_t)n + d] - C[3 * (size_t)o + d])
               : 0.0;
}

// pbar_V = (sum of p over the vertex's active cells) / n_V, w_V = (number of
// its solid cells) / n_V
__global__ void k_vertex_means(int n_nodes, const int* __restrict__ vptr,
                               const int* __restrict__ vcell, const int* __restrict__ active,
                               const double* __restrict__ p, double* __restrict__ pbar,
                               double* __restrict__ w) {
  const int v = blockIdx.x * kBlock + threadIdx.x;
  if (v >= n_nodes) return;
  const int a = vptr[v], e = vptr[v + 1];
  double s = 0.0;
  int solid = 0;
  for (int k = a; k < e; ++k) {
    const int c = vcell[k];
    if (active[c]) s += p[c];
    else ++solid;
  }
  const double inv = e > a ? 1.0 / (double)(e - a) : 0.0;
  pbar[v] = s * inv;
  w[v] = (double)solid * inv;
}

// Masked face gradient (case 3: zero; case 2: solid cells take the mean of
// the face's remaining neighbour cells) and the cross flux x_f = t_f.grad_f;
// GRAD also stores the gradient.
template <bool GRAD>
__global__ void k_face_grad(int n_faces, const int* __restrict__ owner,
                            const int* __restrict__ neigh, const int* __restrict__ active,
                            const int* __restrict__ face_nodes, const int* __restrict__ vptr,
                            const int* __restrict__ vcell, const double* __restrict__ gi,
                            const double* __restrict__ pbar, const double* __restrict__ w,
                            const double* __restrict__ p, const double* __restrict__ t,
                            double* __restrict__ grad, double* __restrict__ xf) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  const int o = owner[f], n = neigh[f];
  double g[3] = {0.0, 0.0, 0.0};
  double x = 0.0;
  if (open_face(active, o, n)) {
    int vv[4];
    double pb[4], wv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      vv[k] = face_nodes[4 * (size_t)f + k];
      pb[k] = pbar[vv[k]];
      wv[k] = w[vv[k]];
    }
    if (wv[0] != 0.0 || wv[1] != 0.0 || wv[2] != 0.0 || wv[3] != 0.0) {
      // mean of p over the distinct active cells of the four vertex lists
      int pos[4], end[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        pos[k] = vptr[vv[k]];
        end[k] = vptr[vv[k] + 1];
      }
      double psum = 0.0;
      int n_act = 0;
      for (;;) {
        int c = INT32_MAX;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (pos[k] < end[k]) c = min(c, vcell[pos[k]]);
        if (c == INT32_MAX) break;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (pos[k] < end[k] && vcell[pos[k]] == c) ++pos[k];
        if (active[c]) {
          psum += p[c];
          ++n_act;
        }
      }
      const double m = psum / (double)n_act;  // the owners are active: n_act >= 2
#pragma unroll
      for (int k = 0; k < 4; ++k) pb[k] += wv[k] * m;
    }
    const double d0 = p[n] - p[o], d1 = pb[2] - pb[0], d2 = pb[3] - pb[1];
#pragma unroll
    for (int d = 0; d < 3; ++d)
      g[d] = gi[(size_t)d * n_faces + f] * d0 + gi[(size_t)(3 + d) * n_faces + f] * d1 +
             gi[(size_t)(6 + d) * n_faces + f] * d2;
#pragma unroll
    for (int d = 0; d < 3; ++d) x += t[(size_t)d * n_faces + f] * g[d];
  }
  if (GRAD) {
#pragma unroll
    for (int d = 0; d < 3; ++d) grad[3 * (size_t)f + d] = g[d];
  }
  xf[f] = x;
}

// ---- cross flux inside a projection: the mask is fixed, and every field
// passed is zero on removed cells ----
enum FaceKind : unsigned char { FK_CLOSED = 0, FK_OPEN = 1, FK_SMEAR = 2 };

// w_V = share of solid cells at vertex V (the mask's part of the means)
__global__ void k_vertex_solid(int n_nodes, const int* __restrict__ vptr,
                               const int* __restrict__ vcell, const int* __restrict__ active,
                               double* __restrict__ w) {
  const int v = blockIdx.x * kBlock + threadIdx.x;
  if (v >= n_nodes) return;
  const int a = vptr[v], e = vptr[v + 1];
  int solid = 0;
  for (int k = a; k < e; ++k) solid += active[vcell[k]] ? 0 : 1;
  w[v] = e > a ? (double)solid / (double)(e - a) : 0.0;
}

// closed (case 3 or wall), open with no solid neighbour (case 1), open with
// solid neighbours (case 2); the cross weights t_f . g_k of open faces
__global__ void k_face_kind(int n_faces, const int* __restrict__ owner,
                            const int* __restrict__ neigh, const int* __restrict__ active,
                            const int* __restrict__ face_nodes, const double* __restrict__ w,
                            const double* __restrict__ gi, const double* __restrict__ t,
                            unsigned char* __restrict__ kind, double* __restrict__ ax) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  const int o = owner[f], n = neigh[f];
  unsigned char k = FK_CLOSED;
  double a[3] = {0.0, 0.0, 0.0};
  if (open_face(active, o, n)) {
    bool sm = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) sm = sm || w[face_nodes[4 * (size_t)f + q]] != 0.0;
    k = sm ? FK_SMEAR : FK_OPEN;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int d = 0; d < 3; ++d)
        a[c] += t[(size_t)d * n_faces + f] * gi[(size_t)(3 * c + d) * n_faces + f];
  }
  kind[f] = k;
#pragma unroll
  for (int c = 0; c < 3; ++c) ax[(size_t)c * n_faces + f] = a[c];
}

// pbar_V = (sum of p over the vertex's cells) / n_V; p is zero on removed
// cells, so this is the active-cell sum of the masked means
// A vertex's cells are requested kVertexU at a time, then their values, and
// added in the list's order: one by one the loop was a chain of dependent
// loads (275 k vertices 9.6 -> 8.4 us).
constexpr int kVertexU = 8;

__global__ void k_vertex_sum(int n_nodes, const int* __restrict__ vptr,
                             const int* __restrict__ vcell, const double* __restrict__ p,
                             double* __restrict__ pbar) {
  const int v = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (v >= n_nodes) return;
  const int a = vptr[v], e = vptr[v + 1];
  double s = 0.0;
  for (int k = a; k < e; k += kVertexU) {
    int c[kVertexU];
    double g[kVertexU];
#pragma unroll
    for (int u = 0; u < kVertexU; ++u) c[u] = k + u < e ? vcell[k + u] : -1;
#pragma unroll
    for (int u = 0; u < kVertexU; ++u) g[u] = c[u] >= 0 ? p[c[u]] : 0.0;
#pragma unroll
    for (int u = 0; u < kVertexU; ++u)
      if (c[u] >= 0) s += g[u];
  }
  pbar[v] = e > a ? s / (double)(e - a) : 0.0;
}

// x_f = t_f . grad(p)_f = sum_k a_k(f) d_k on open faces without solid
// neighbours (case 1), 0 on closed faces; case-2 faces are left to
// k_face_cross_smear, so that these waves stay uniform.
__global__ void k_face_cross(int n_faces, const int* __restrict__ owner,
                             const int* __restrict__ neigh, const int* __restrict__ face_nodes,
                             const unsigned char* __restrict__ kind, const double* __restrict__ ax,
                             const double* __restrict__ pbar, const double* __restrict__ p,
                             double* __restrict__ xf) {
  const int f = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  const unsigned char k = kind[f];
  if (k == FK_SMEAR) return;
  double x = 0.0;
  if (k == FK_OPEN) {
    const int o = owner[f], n = neigh[f];
    const int4 vv = *reinterpret_cast<const int4*>(face_nodes + 4 * (size_t)f);
    x = ax[f] * (p[n] - p[o]) + ax[(size_t)n_faces + f] * (pbar[vv.z] - pbar[vv.x]) +
        ax[2 * (size_t)n_faces + f] * (pbar[vv.w] - pbar[vv.y]);
  }
  xf[f] = x;
}

// Distinct active cells among the four vertex lists of face f (the cells
// whose mean replaces the solid ones, Eq. 15-16), in ascending order: the
// count (cells == nullptr) or the cells themselves.
__device__ __forceinline__ int smear_cells(int f, const int* __restrict__ active,
                                           const int* __restrict__ face_nodes,
                                           const int* __restrict__ vptr,
                                           const int* __restrict__ vcell, int* __restrict__ cells) {
  int pos[4], end[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int v = face_nodes[4 * (size_t)f + q];
    pos[q] = vptr[v];
    end[q] = vptr[v + 1];
  }
  int n_act = 0;
  for (;;) {
    int c = INT32_MAX;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (pos[q] < end[q]) c = min(c, vcell[pos[q]]);
    if (c == INT32_MAX) break;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (pos[q] < end[q] && vcell[pos[q]] == c) ++pos[q];
    if (active[c]) {
      if (cells) cells[n_act] = c;
      ++n_act;
    }
  }
  return n_act;
}

// once per projection: count[f] = that number on case-2 faces, 0 elsewhere
__global__ void k_smear_count(int n_faces, const unsigned char* __restrict__ kind,
                              const int* __restrict__ active, const int* __restrict__ face_nodes,
                              const int* __restrict__ vptr, const int* __restrict__ vcell,
                              int* __restrict__ count) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  count[f] = kind[f] == FK_SMEAR ? smear_cells(f, active, face_nodes, vptr, vcell, nullptr) : 0;
}

__global__ void k_smear_fill(const long long* __restrict__ n_list, const int* __restrict__ list,
                             const int* __restrict__ active, const int* __restrict__ face_nodes,
                             const int* __restrict__ vptr, const int* __restrict__ vcell,
                             const int* __restrict__ off, int* __restrict__ cells) {
  const long long nl = *n_list;
  for (long long i = blockIdx.x * (long long)kBlock + threadIdx.x; i < nl;
       i += (long long)gridDim.x * kBlock) {
    const int f = list[i];
    smear_cells(f, active, face_nodes, vptr, vcell, cells + off[f]);
  }
}

// Case-2 faces (listed, *n_list of them): the solid cells of the four vertex
// means take the mean m of the face's remaining neighbour cells, whose
// ascending list cells[off[f]..off[f+1]) was built for this mask.  kSmearLanes
// lanes share a list (8 to 18 cells): a thread per list was a chain of as many
// dependent gathers over too few wavefronts (a 64^3 front: 14.1 -> 6.0 us).
constexpr int kSmearLanes = 8;

__global__ void k_face_cross_smear(const long long* __restrict__ n_list,
                                   const int* __restrict__ list, int n_faces,
                                   const int* __restrict__ owner, const int* __restrict__ neigh,
                                   const int* __restrict__ face_nodes,
                                   const int* __restrict__ off, const int* __restrict__ cells,
                                   const double* __restrict__ ax, const double* __restrict__ pbar,
                                   const double* __restrict__ w, const double* __restrict__ p,
                                   double* __restrict__ xf) {
  const long long nl = *n_list;
  const int l = threadIdx.x % kSmearLanes;
  constexpr int kPer = kBlock / kSmearLanes;
  for (long long i = blockIdx.x * (long long)kPer + threadIdx.x / kSmearLanes; i < nl;
       i += (long long)gridDim.x * kPer) {
    const int f = list[i];
    const int a = off[f], e = off[f + 1];
    double psum = 0.0;
    for (int k = a + l; k < e; k += kSmearLanes) psum += p[cells[k]];
#pragma unroll
    for (int q = kSmearLanes / 2; q > 0; q >>= 1) psum += __shfl_down(psum, q, kSmearLanes);
    if (l != 0) continue;
    const int o = owner[f], n = neigh[f];
    const double m = psum / (double)(e - a);  // the owners are active: e - a >= 2
    const int4 vv = *reinterpret_cast<const int4*>(face_nodes + 4 * (size_t)f);
    const double pb0 = pbar[vv.x] + w[vv.x] * m, pb1 = pbar[vv.y] + w[vv.y] * m;
    const double pb2 = pbar[vv.z] + w[vv.z] * m, pb3 = pbar[vv.w] + w[vv.w] * m;
    xf[f] = ax[f] * (p[n] - p[o]) + ax[(size_t)n_faces + f] * (pb2 - pb0) +
            ax[2 * (size_t)n_faces + f] * (pb3 - pb1);
  }
}

__global__ void k_smear_flags(int n_faces, const unsigned char* __restrict__ kind,
                              int* __restrict__ flag) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f < n_faces) flag[f] = kind[f] == FK_SMEAR ? 1 : 0;
}

__global__ void k_set_last(const long long* __restrict__ v, int* __restrict__ dst) {
  *dst = (int)*v;
}

__global__ void k_smear_list(int n_faces, const unsigned char* __restrict__ kind,
                             const int* __restrict__ pos, int* __restrict__ list) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f < n_faces && kind[f] == FK_SMEAR) list[pos[f]] = f;
}

// r = b + X p - L p on non-pinned active cells (0 elsewhere), with block
// partials of r.r
__global__ void __launch_bounds__(kBlock) k_full_residual(
    int n_cells, const int* __restrict__ adj_ptr, const int* __restrict__ adj_nbr,
    const int* __restrict__ adj_face, const int* __restrict__ owner,
    const int* __restrict__ active, const int* __restrict__ comp, const double* __restrict__ coeff,
    const double* __restrict__ b, const double* __restrict__ xf, const double* __restrict__ p,
    double* __restrict__ r, double* __restrict__ part) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  double v = 0.0;
  if (c < n_cells) {
    if (active[c] && comp[c] != c) {
      const double pc = p[c];
      double s = b[c];
      for (int e = adj_ptr[c]; e < adj_ptr[c + 1]; ++e) {
        const int nb = adj_nbr[e];
        if (!active[nb]) continue;
        const int f = adj_face[e];
        s += (owner[f] == c ? xf[f] : -xf[f]) - coeff[f] * (pc - p[nb]);
      }
      v = s;
    }
    r[c] = v;
  }
  v = block_sum<kBlock>(v * v);
  if (threadIdx.x == 0) part[blockIdx.x] = v;
}

// sum of the first n partials in index order
__global__ void __launch_bounds__(kBlock) k_sum_partials(const double* __restrict__ part, int n,
                                                         double* __restrict__ out) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += kBlock) s += part[i];
  s = block_sum<kBlock>(s);
  if (threadIdx.x == 0) *out = s;
}

// warm start: p = 0 on removed cells and pins (kept elsewhere); block
// partials of b.b over the non-pinned active cells
__global__ void __launch_bounds__(kBlock) k_clean_start(int n, const int* __restrict__ active,
                                                        const int* __restrict__ comp,
                                                        const double* __restrict__ b,
                                                        double* __restrict__ p,
                                                        double* __restrict__ part) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  double v = 0.0;
  if (c < n) {
    const bool free = active[c] && comp[c] != c;
    if (!free) p[c] = 0.0;
    v = free ? b[c] * b[c] : 0.0;
  }
  v = block_sum<kBlock>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v;
}

__global__ void k_add_cells(int n, const double* __restrict__ d, double* __restrict__ p) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c < n) p[c] += d[c];
}

// Eq. 17 on open faces, 0 on blocked and wall faces
__global__ void k_corrected_flux(int n_faces, const int* __restrict__ owner,
                                 const int* __restrict__ neigh, const int* __restrict__ active,
                                 const double* __restrict__ Fs, const double* __restrict__ coeff,
                                 const double* __restrict__ p, const double* __restrict__ xf,
                                 double dt, double* __restrict__ F) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= n_faces) return;
  const int o = owner[f], n = neigh[f];
  F[f] = open_face(active, o, n) ? Fs[f] - dt * (coeff[f] * (p[n] - p[o]) + xf[f]) : 0.0;
}

// Eq. 8 with the cell gradient the mean of the open faces' gradients; u* on
// an active cell without open faces, 0 on removed cells
__global__ void k_corrected_velocity(int n_cells, const int* __restrict__ adj_ptr,
                                     const int* __restrict__ adj_nbr,
                                     const int* __restrict__ adj_face,
                                     const int* __restrict__ active,
                                     const double* __restrict__ grad,
                                     const double* __restrict__ ustar, double dt_rho,
                                     double* __restrict__ u) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= n_cells) return;
  double out[3] = {0.0, 0.0, 0.0};
  if (active[c]) {
    double g[3] = {0.0, 0.0, 0.0};
    int k = 0;
    for (int e = adj_ptr[c]; e < adj_ptr[c + 1]; ++e) {
      if (!active[adj_nbr[e]]) continue;
      const int f = adj_face[e];
#pragma unroll
      for (int d = 0; d < 3; ++d) g[d] += grad[3 * (size_t)f + d];
      ++k;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d)
      out[d] = ustar[3 * (size_t)c + d] - (k ? dt_rho * g[d] / (double)k : 0.0);
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) u[3 * (size_t)c + d] = out[d];
}

// ---- BiCGSTAB on (L - X) p = b' (the cross term implicit) ----
// Vectors are indexed by cell and zero on removed cells and pins.  The
// scalars of iteration i (counted from the last restart) live in
// sc[kSc * i + k]: r^.r at its start, r.r, alpha, omega.
constexpr int kSc = 4;
enum { SC_RHO = 0, SC_RR = 1, SC_ALPHA = 2, SC_OMEGA = 3 };
constexpr int kBicgRestart = 200;  // iterations before a forced restart

__global__ void k_gather_free(int na, const int* __restrict__ perm, const int* __restrict__ comp,
                              const double* __restrict__ y, double* __restrict__ yc) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= na) return;
  const int c = perm[r];
  yc[r] = comp[c] == c ? 0.0 : y[c];
}

__global__ void k_scatter_free(int nc, const int* __restrict__ cid, const int* __restrict__ comp,
                               const double* __restrict__ zc, double* __restrict__ z) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= nc) return;
  const int k = cid[c];
  z[c] = (k < 0 || comp[c] == c) ? 0.0 : zc[k];
}

// out = L y - X y on non-pinned active cells (0 elsewhere), with block
// partials of w.out (and of out.out for TWO) in part[0..G) and part[G..2G).
// The operands of kApplyU faces are requested before the first is used and
// added in the faces' order (64^3: 11.8 -> 9.7 us).
constexpr int kApplyU = 6;

template <bool TWO>
__global__ void __launch_bounds__(kBlock) k_apply_full(
    int n_cells, const int* __restrict__ adj_ptr, const int* __restrict__ adj_nbr,
    const int* __restrict__ adj_face, const int* __restrict__ owner,
    const int* __restrict__ active, const int* __restrict__ comp, const double* __restrict__ coeff,
    const double* __restrict__ xf, const double* __restrict__ y, const double* __restrict__ w,
    double* __restrict__ out, double* __restrict__ part) {
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  const int c = blk * kBlock + threadIdx.x;
  double v = 0.0, wv = 0.0;
  if (c < n_cells) {
    if (active[c] && comp[c] != c) {
      const double yc = y[c];
      double acc = 0.0;
      const int e0 = adj_ptr[c], e1 = adj_ptr[c + 1];
      for (int e = e0; e < e1; e += kApplyU) {
        int nb[kApplyU], f[kApplyU], on[kApplyU];
        double k[kApplyU], yn[kApplyU], x[kApplyU];
#pragma unroll
        for (int u = 0; u < kApplyU; ++u) {
          nb[u] = e + u < e1 ? adj_nbr[e + u] : c;
          f[u] = e + u < e1 ? adj_face[e + u] : -1;
        }
#pragma unroll
        for (int u = 0; u < kApplyU; ++u) {
          const int g = f[u] >= 0 ? f[u] : 0;
          on[u] = f[u] >= 0 && active[nb[u]];
          yn[u] = y[nb[u]];
          k[u] = coeff[g];
          x[u] = owner[g] == c ? xf[g] : -xf[g];
        }
#pragma unroll
        for (int u = 0; u < kApplyU; ++u)
          if (on[u]) acc += k[u] * (yc - yn[u]) - x[u];
      }
      v = acc;
      wv = w[c] * v;
    }
    out[c] = v;
  }
  wv = block_sum<kBlock>(wv);
  if (threadIdx.x == 0) part[blk] = wv;
  if (TWO) {
    v = block_sum<kBlock>(v * v);
    if (threadIdx.x == 0) part[gridDim.x + blk] = v;
  }
}

// One workgroup: MODE 0 alpha_i = rho_i / (r^.v); MODE 1 omega_i =
// (t.s)/(t.t); MODE 2 rho_(i+1) = r^.r, rr_(i+1) = r.r; MODE 3 (restart)
// rho_0 = rr_0 = the value at src.
template <int MODE>
__global__ void __launch_bounds__(kBlock) k_bicg_scalar(int G, const double* __restrict__ part,
                                                        double* __restrict__ sc, int i,
                                                        const double* __restrict__ src) {
  double a = 0.0, b = 0.0;
  if (MODE != 3) {
    for (int k = threadIdx.x; k < G; k += kBlock) a += part[k];
    a = block_sum<kBlock>(a);
    if (MODE != 0) {
      for (int k = threadIdx.x; k < G; k += kBlock) b += part[G + k];
      b = block_sum<kBlock>(b);
    }
  }
  if (threadIdx.x != 0) return;
  double* cur = sc + (size_t)kSc * i;
  if (MODE == 0) cur[SC_ALPHA] = cur[SC_RHO] / a;
  if (MODE == 1) cur[SC_OMEGA] = b > 0.0 ? a / b : 0.0;
  if (MODE == 2) {
    cur[kSc + SC_RHO] = a;
    cur[kSc + SC_RR] = b;
  }
  if (MODE == 3) {
    cur[SC_RHO] = *src;
    cur[SC_RR] = *src;
  }
}

// search direction: p = r on the first iteration, else
// p = r + beta (p - omega v), beta = (rho_i / rho_(i-1)) (alpha / omega)_(i-1)
__global__ void k_bicg_dir(int nc, const double* __restrict__ r, const double* __restrict__ v,
                           double* __restrict__ pp, const double* __restrict__ sc, int i) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= nc) return;
  if (i == 0) {
    pp[c] = r[c];
    return;
  }
  const double* prev = sc + (size_t)kSc * (i - 1);
  const double* cur = prev + kSc;
  const double beta = (cur[SC_RHO] / prev[SC_RHO]) * (prev[SC_ALPHA] / prev[SC_OMEGA]);
  pp[c] = r[c] + beta * (pp[c] - prev[SC_OMEGA] * v[c]);
}

__global__ void k_bicg_s(int nc, const double* __restrict__ r, const double* __restrict__ v,
                         double* __restrict__ sv, const double* __restrict__ sc, int i) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c < nc) sv[c] = r[c] - sc[(size_t)kSc * i + SC_ALPHA] * v[c];
}

// x += alpha y + omega z; r = s - omega t; partials of r^.r and r.r
__global__ void __launch_bounds__(kBlock) k_bicg_xr(
    int nc, double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ sv, const double* __restrict__ tv, double* __restrict__ r,
    const double* __restrict__ rh, const double* __restrict__ sc, int i, double* __restrict__ part) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  const double alpha = sc[(size_t)kSc * i + SC_ALPHA], omega = sc[(size_t)kSc * i + SC_OMEGA];
  double a = 0.0, b = 0.0;
  if (c < nc) {
    x[c] += alpha * y[c] + omega * z[c];
    const double rc = sv[c] - omega * tv[c];
    r[c] = rc;
    a = rh[c] * rc;
    b = rc * rc;
  }
  a = block_sum<kBlock>(a);
  b = block_sum<kBlock>(b);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = a;
    part[gridDim.x + blockIdx.x] = b;
  }
}

struct RtolGuard {
  ppe_solver* s;
  double saved;
  RtolGuard(ppe_solver* s_, double v) : s(s_), saved(s_->opt.rtol) { s->opt.rtol = v; }
  ~RtolGuard() { s->opt.rtol = saved; }
};

}  // namespace

void set_geometry(ppe_solver* s, int n_nodes, const double* nodes, const int32_t* face_nodes,
                  const int32_t* cell_nodes, const double* cell_centre, const double* face_area) {
  const int nc = s->n_cells, nf = s->n_faces;
  s->geom_ok = false;
  s->n_nodes = n_nodes;
  double* X = s->g_nodes.get<double>(3 * (size_t)n_nodes);
  double* C = s->g_cc.get<double>(3 * (size_t)nc);
  double* S = s->g_S.get<double>(3 * (size_t)nf);
  int* fnodes = s->g_fnodes.get<int>(4 * (size_t)nf);
  int* cnodes = s->tmp_i[2].get<int>(8 * (size_t)nc);
  PPE_HIP(hipMemcpyAsync(X, nodes, sizeof(double) * 3 * n_nodes, hipMemcpyDeviceToDevice, s->stream));
  PPE_HIP(hipMemcpyAsync(C, cell_centre, sizeof(double) * 3 * nc, hipMemcpyDeviceToDevice, s->stream));
  if (nf) {
    PPE_HIP(hipMemcpyAsync(S, face_area, sizeof(double) * 3 * nf, hipMemcpyDeviceToDevice, s->stream));
    PPE_HIP(hipMemcpyAsync(fnodes, face_nodes, sizeof(int) * 4 * nf, hipMemcpyDeviceToDevice,
                           s->stream));
  }
  PPE_HIP(hipMemcpyAsync(cnodes, cell_nodes, sizeof(int) * 8 * nc, hipMemcpyDeviceToDevice,
                         s->stream));
  int* flag = s->flag.get<int>(kFlagWords);
  fill_int(s, flag, 0, 1);
  // vertex -> cells
  int* vcnt = s->tmp_i[0].get<int>(n_nodes + 1);
  fill_int(s, vcnt, 0, n_nodes + 1);
  hipLaunchKernelGGL(k_vertex_count, dim3(grid_for(nc)), dim3(kBlock), 0, s->stream, nc, n_nodes,
                     cnodes, vcnt, flag);
  PPE_LAUNCH_CHECK();
  require(read_scalar(s, flag) == 0, PPE_ERR_ARG,
          "cell_nodes: a vertex index out of range or repeated within a cell");
  int* vptr = s->g_vptr.get<int>(n_nodes + 1);
  const long long nvc = exclusive_scan(s, vcnt, vptr, n_nodes);
  int* cursor = s->tmp_i[1].get<int>(n_nodes + 1);
  PPE_HIP(hipMemcpyAsync(cursor, vptr, sizeof(int) * (n_nodes + 1), hipMemcpyDeviceToDevice,
                         s->stream));
  int* vcell = s->g_vcell.get<int>(nvc);
  hipLaunchKernelGGL(k_vertex_fill, dim3(grid_for(nc)), dim3(kBlock), 0, s->stream, nc, cnodes,
                     cursor, vcell);
  PPE_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_vertex_sort, dim3(grid_for(n_nodes)), dim3(kBlock), 0, s->stream, n_nodes,
                     vptr, vcell, flag);
  PPE_LAUNCH_CHECK();
  // local frames
  double* gi = s->g_inv.get<double>(9 * (size_t)(nf > 0 ? nf : 1));
  if (nf) {
    hipLaunchKernelGGL(k_face_frame, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf, n_nodes,
                       s->owner.as<int>(), s->neigh.as<int>(), fnodes, vptr, vcell, X, C, gi, flag);
    PPE_LAUNCH_CHECK();
  }
  const int bits = read_scalar(s, flag);
  require(!(bits & GE_VALENCE), PPE_ERR_ARG, "a vertex is shared by more than 16 cells");
  require(!(bits & GE_INDEX), PPE_ERR_ARG, "face_nodes: a vertex index out of range");
  require(!(bits & GE_CORNER), PPE_ERR_ARG,
          "a face's vertices are not corners of both of its cells");
  require(!(bits & GE_SINGULAR), PPE_ERR_ARG,
          "a face's local frame (C1C2, V1V3, V2V4) is singular");
  s->geom_ok = true;
}

void cross_vectors(ppe_solver* s, const double* coeff, double rho, double* t) {
  const int nf = s->n_faces;
  if (nf == 0) return;
  hipLaunchKernelGGL(k_cross_vectors, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf,
                     s->owner.as<int>(), s->neigh.as<int>(), s->g_S.as<double>(),
                     s->g_cc.as<double>(), coeff, 1.0 / rho, t);
  PPE_LAUNCH_CHECK();
}

void face_gradient(ppe_solver* s, const double* p, const double* t, double* grad, double* xf) {
  const int nf = s->n_faces, nn = s->n_nodes;
  if (nf == 0) return;
  double* pbar = s->pj_vm.get<double>(2 * (size_t)nn);
  double* w = pbar + nn;
  hipLaunchKernelGGL(k_vertex_means, dim3(grid_for(nn)), dim3(kBlock), 0, s->stream, nn,
                     s->g_vptr.as<int>(), s->g_vcell.as<int>(), s->active.as<int>(), p, pbar, w);
  PPE_LAUNCH_CHECK();
#define PPE_FACE_GRAD(G_)                                                                      \
  hipLaunchKernelGGL(k_face_grad<G_>, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf,         \
                     s->owner.as<int>(), s->neigh.as<int>(), s->active.as<int>(),                 \
                     s->g_fnodes.as<int>(), s->g_vptr.as<int>(), s->g_vcell.as<int>(),            \
                     s->g_inv.as<double>(), pbar, w, p, t, grad, xf)
  if (grad) PPE_FACE_GRAD(true);
  else PPE_FACE_GRAD(false);
#undef PPE_FACE_GRAD
  PPE_LAUNCH_CHECK();
}

namespace {

// Mask-dependent face data of one projection: solid shares, face kinds and
// the cross weights of the cross vectors t.
struct CrossData {
  unsigned char* kind;
  double* ax;
  double* w;
  double* pbar;
  int* list;               // case-2 faces
  const long long* count;  // their number (device)
  int* off;                // their remaining cells: cells[off[f]..off[f+1])
  int* cells;
};

CrossData prepare_cross(ppe_solver* s, const double* t) {
  const int nf = s->n_faces, nn = s->n_nodes;
  CrossData cd{};
  cd.w = s->pj_vm.get<double>(2 * (size_t)nn);
  cd.pbar = cd.w + nn;
  cd.ax = s->pj_ax.get<double>(3 * (size_t)(nf > 0 ? nf : 1));
  cd.kind = s->pj_kind.get<unsigned char>(nf > 0 ? nf : 1);
  hipLaunchKernelGGL(k_vertex_solid, dim3(grid_for(nn)), dim3(kBlock), 0, s->stream, nn,
                     s->g_vptr.as<int>(), s->g_vcell.as<int>(), s->active.as<int>(), cd.w);
  PPE_LAUNCH_CHECK();
  if (nf == 0) return cd;
  const int* active = s->active.as<int>();
  const int* fnodes = s->g_fnodes.as<int>();
  const int* vptr = s->g_vptr.as<int>();
  const int* vcell = s->g_vcell.as<int>();
  hipLaunchKernelGGL(k_face_kind, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf,
                     s->owner.as<int>(), s->neigh.as<int>(), active, fnodes, cd.w,
                     s->g_inv.as<double>(), t, cd.kind, cd.ax);
  PPE_LAUNCH_CHECK();
  // the case-2 faces: a list, and for each the ascending list of its
  // remaining neighbour cells
  int* buf = s->pj_list.get<int>(4 * (size_t)nf + 4);
  int* flag = buf;
  int* pos = flag + nf + 1;
  int* cnt = pos + nf + 1;
  cd.off = cnt + nf + 1;
  hipLaunchKernelGGL(k_smear_flags, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf, cd.kind,
                     flag);
  PPE_LAUNCH_CHECK();
  const long long* total = exclusive_scan_async(s, flag, pos, nf, 0);
  long long* counts = s->pj_cnt.get<long long>(2);
  // the scan totals sit in shared slots: keep copies of our own
  PPE_HIP(hipMemcpyAsync(counts, total, sizeof(long long), hipMemcpyDeviceToDevice, s->stream));
  cd.count = counts;
  cd.list = flag;  // the flags are consumed by the scan; the list reuses them
  hipLaunchKernelGGL(k_smear_list, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf, cd.kind,
                     pos, cd.list);
  PPE_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_smear_count, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf, cd.kind,
                     active, fnodes, vptr, vcell, cnt);
  PPE_LAUNCH_CHECK();
  const long long* nnz_d = exclusive_scan_async(s, cnt, cd.off, nf, 1);
  long long nnz = 0;
  read_back(s, {ReadItem{nnz_d, sizeof(long long), &nnz}});
  // off[nf] = nnz closes the last row
  PPE_HIP(hipMemcpyAsync(counts + 1, nnz_d, sizeof(long long), hipMemcpyDeviceToDevice, s->stream));
  hipLaunchKernelGGL(k_set_last, dim3(1), dim3(1), 0, s->stream, counts + 1, cd.off + nf);
  PPE_LAUNCH_CHECK();
  cd.cells = s->pj_cells.get<int>(nnz > 0 ? (size_t)nnz : 1);
  const int gs = grid_for(nf) < 512 ? grid_for(nf) : 512;
  hipLaunchKernelGGL(k_smear_fill, dim3(gs), dim3(kBlock), 0, s->stream, cd.count, cd.list, active,
                     fnodes, vptr, vcell, cd.off, cd.cells);
  PPE_LAUNCH_CHECK();
  return cd;
}

// xf = t_f . grad(p)_f for a field p that is zero on removed cells
void cross_flux(ppe_solver* s, const CrossData& cd, const double* p, double* xf) {
  const int nf = s->n_faces, nn = s->n_nodes;
  if (nf == 0) return;
  hipLaunchKernelGGL(k_vertex_sum, dim3(grid_for(nn)), dim3(kBlock), 0, s->stream, nn,
                     s->g_vptr.as<int>(), s->g_vcell.as<int>(), p, cd.pbar);
  PPE_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_face_cross, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf,
                     s->owner.as<int>(), s->neigh.as<int>(), s->g_fnodes.as<int>(), cd.kind,
                     cd.ax, cd.pbar, p, xf);
  PPE_LAUNCH_CHECK();
  const int gs = grid_for(nf) < 512 ? grid_for(nf) : 512;
  hipLaunchKernelGGL(k_face_cross_smear, dim3(gs), dim3(kBlock), 0, s->stream, cd.count, cd.list,
                     nf, s->owner.as<int>(), s->neigh.as<int>(), s->g_fnodes.as<int>(), cd.off,
                     cd.cells, cd.ax, cd.pbar, cd.w, p, xf);
  PPE_LAUNCH_CHECK();
}

}  // namespace

ppe_status project(ppe_solver* s, const double* coeff, const double* ustar, double rho, double dt,
                   double* p, double* flux, double* u, ppe_project_stats* out, bool use_x0) {
  const int nc = s->n_cells, nf = s->n_faces;
  ppe_project_stats st{};
  const int* owner = s->owner.as<int>();
  const int* neigh = s->neigh.as<int>();
  const int* active = s->active.as<int>();
  const int* aptr = s->adj_ptr.as<int>();
  const int* anbr = s->adj_nbr.as<int>();
  const int* aface = s->adj_face.as<int>();
  double* Fs = s->pj_fs.get<double>(nf > 0 ? nf : 1);
  double* b = s->pj_b.get<double>(nc);
  double* r = s->pj_r.get<double>(nc);
  double* delta = s->pj_d.get<double>(nc);
  double* grad = s->pj_grad.get<double>(3 * (size_t)(nf > 0 ? nf : 1));
  double* xf = s->pj_xf.get<double>(nf > 0 ? nf : 1);
  const int gc = grid_for(nc);
  double* part = s->pj_part.get<double>(gc + 3);
  double* sums = part + gc;  // [0] r.r at the start, [1] r.r, [2] b.b (warm start)
  if (nf) {
    hipLaunchKernelGGL(k_star_flux, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf, owner,
                       neigh, active, ustar, s->g_S.as<double>(), Fs);
    PPE_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(k_rhs_from_flux, dim3(gc), dim3(kBlock), 0, s->stream, nc, aptr, anbr, aface,
                     owner, active, Fs, 1.0 / dt, b);
  PPE_LAUNCH_CHECK();
  double* t = s->pj_t.get<double>(3 * (size_t)(nf > 0 ? nf : 1));
  cross_vectors(s, coeff, rho, t);
  const CrossData cd = prepare_cross(s, t);
  double bn_warm = 0.0;
  if (use_x0) {
    // the given pressure, zero on removed cells and pins, and the reference
    // ||b'|| of the pinned right-hand side
    hipLaunchKernelGGL(k_clean_start, dim3(gc), dim3(kBlock), 0, s->stream, nc, active,
                       s->comp_full.as<int>(), b, p, part);
    PPE_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, s->stream, part, gc, sums + 2);
    PPE_LAUNCH_CHECK();
    read_back(s, {ReadItem{sums + 2, sizeof(double), &bn_warm}});
    bn_warm = std::sqrt(bn_warm);
    if (!(bn_warm > 0.0)) fill_double(s, p, 0.0, nc);  // b' = 0: p = 0 solves it
  } else {
    fill_double(s, p, 0.0, nc);
  }
  // r = b + X p - L p; at p = 0 it is b on the non-pinned active cells, whose
  // norm is the reference ||b'||
  auto residual = [&](int slot) {
    cross_flux(s, cd, p, xf);
    hipLaunchKernelGGL(k_full_residual, dim3(gc), dim3(kBlock), 0, s->stream, nc, aptr, anbr, aface,
                       owner, active, s->comp_full.as<int>(), coeff, b, xf, p, r, part);
    PPE_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, s->stream, part, gc, sums + slot);
    PPE_LAUNCH_CHECK();
    double v = 0.0;
    read_back(s, {ReadItem{sums + slot, sizeof(double), &v}});
    return std::sqrt(v);
  };
  double rn = residual(0);
  const double bn = use_x0 ? bn_warm : rn;
  // one decade below rtol: loose inner solves leave the last residual in
  // smooth modes, which the condition number amplifies in the pressure; the
  // margin keeps p near the exact solution of the full system at the price
  // of about one pass
  const double target = 0.1 * s->opt.rtol * bn;
  ppe_status status = PPE_OK;
  if (s->opt.project_krylov == 1 && rn > target) {
    // BiCGSTAB, right-preconditioned by one V-cycle of L per application.
    // On breakdown or at the iteration cap the deferred correction below
    // takes over from the current iterate.
    const int na = s->n_active;
    double* kv = s->pj_k.get<double>(7 * (size_t)nc + 2 * (size_t)(na > 0 ? na : 1) +
                                     2 * (size_t)gc + (size_t)kSc * (kBicgRestart + 2));
    double* rh = kv;
    double* pp = rh + nc;
    double* v = pp + nc;
    double* sv = v + nc;
    double* tv = sv + nc;
    double* y = tv + nc;
    double* z = y + nc;
    double* yc = z + nc;
    double* zc = yc + (na > 0 ? na : 1);
    double* bpart = zc + (na > 0 ? na : 1);  // 2 gc block partials
    double* sc = bpart + 2 * (size_t)gc;
    const int* perm = s->perm.as<int>();
    const int* cid = s->cid.as<int>();
    const int* comp = s->comp_full.as<int>();
    const int ga = grid_for(na);
    auto precond = [&](const double* in, double* outv) {
      hipLaunchKernelGGL(k_gather_free, dim3(ga), dim3(kBlock), 0, s->stream, na, perm, comp, in, yc);
      PPE_LAUNCH_CHECK();
      vcycle(s, 0, yc, zc);
      hipLaunchKernelGGL(k_scatter_free, dim3(gc), dim3(kBlock), 0, s->stream, nc, cid, comp, zc,
                         outv);
      PPE_LAUNCH_CHECK();
    };
    auto apply = [&](const double* in, const double* w, double* outv, bool two) {
      cross_flux(s, cd, in, xf);
      if (two)
        hipLaunchKernelGGL(k_apply_full<true>, dim3(gc), dim3(kBlock), 0, s->stream, nc, aptr, anbr,
                           aface, owner, active, comp, coeff, xf, in, w, outv, bpart);
      else
        hipLaunchKernelGGL(k_apply_full<false>, dim3(gc), dim3(kBlock), 0, s->stream, nc, aptr,
                           anbr, aface, owner, active, comp, coeff, xf, in, w, outv, bpart);
      PPE_LAUNCH_CHECK();
    };
    bool done = false, broke = false;
    bool fresh = true;  // r is a true residual and sums[slot] its r.r
    int slot = 0;
    while (!done && !broke && st.outer < s->opt.max_iter) {
      if (!fresh) {
        rn = residual(1);
        slot = 1;
        if (rn <= target) {
          done = true;
          break;
        }
      }
      fresh = false;
      // (re)start from the true residual: r^ = r
      PPE_HIP(hipMemcpyAsync(rh, r, sizeof(double) * nc, hipMemcpyDeviceToDevice, s->stream));
      hipLaunchKernelGGL(k_bicg_scalar<3>, dim3(1), dim3(kBlock), 0, s->stream, 0, bpart, sc, 0,
                         sums + slot);
      PPE_LAUNCH_CHECK();
      for (int i = 0; i < kBicgRestart && st.outer < s->opt.max_iter; ++i) {
        hipLaunchKernelGGL(k_bicg_dir, dim3(gc), dim3(kBlock), 0, s->stream, nc, r, v, pp, sc, i);
        PPE_LAUNCH_CHECK();
        precond(pp, y);
        apply(y, rh, v, false);
        hipLaunchKernelGGL(k_bicg_scalar<0>, dim3(1), dim3(kBlock), 0, s->stream, gc, bpart, sc, i,
                           nullptr);
        PPE_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_bicg_s, dim3(gc), dim3(kBlock), 0, s->stream, nc, r, v, sv, sc, i);
        PPE_LAUNCH_CHECK();
        precond(sv, z);
        apply(z, sv, tv, true);
        hipLaunchKernelGGL(k_bicg_scalar<1>, dim3(1), dim3(kBlock), 0, s->stream, gc, bpart, sc, i,
                           nullptr);
        PPE_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_bicg_xr, dim3(gc), dim3(kBlock), 0, s->stream, nc, p, y, z, sv, tv, r,
                           rh, sc, i, bpart);
        PPE_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_bicg_scalar<2>, dim3(1), dim3(kBlock), 0, s->stream, gc, bpart, sc, i,
                           nullptr);
        PPE_LAUNCH_CHECK();
        st.outer += 1;
        st.pcg_iterations += 2;  // V-cycles
        double q[4] = {0.0, 0.0, 0.0, 0.0};  // alpha, omega, rho_(i+1), rr_(i+1)
        read_back(s, {ReadItem{sc + (size_t)kSc * i + SC_ALPHA, sizeof(double) * 2, q},
                      ReadItem{sc + (size_t)kSc * (i + 1), sizeof(double) * 2, q + 2}});
        if (std::isfinite(q[3]) && std::sqrt(q[3]) <= target) {
          // the recursive residual met the target: the true one decides (a
          // miss restarts from it)
          rn = residual(1);
          slot = 1;
          fresh = true;
          done = rn <= target;
          break;
        }
        if (!std::isfinite(q[0]) || !std::isfinite(q[1]) || q[1] == 0.0 || !std::isfinite(q[3]) ||
            q[2] == 0.0) {
          broke = true;
          break;
        }
      }
    }
    if (!done) rn = residual(1);
  }
  const int max_outer = 50;
  int dc_passes = 0;
  while (rn > target) {
    if (dc_passes == max_outer) {
      status = PPE_NOT_CONVERGED;
      break;
    }
    ++dc_passes;
    // correction solve to 5%: the outer contraction is at best the size of
    // L^-1 X (a few percent), so tighter inner solves gain nothing; on the
    // last pass, only as tight as the target needs
    const double inner = std::min(0.5, std::max(0.05, 0.3 * target / rn));
    ppe_status ist;
    {
      RtolGuard g(s, inner);
      ist = pcg_solve(s, r, delta, 0, &s->pred_inner);
    }
    s->solves_since_assemble += 1;
    st.pcg_iterations += s->stats.iterations;
    st.outer += 1;
    if (ist < 0) return ist;
    hipLaunchKernelGGL(k_add_cells, dim3(gc), dim3(kBlock), 0, s->stream, nc, delta, p);
    PPE_LAUNCH_CHECK();
    rn = residual(1);
  }
  st.rel_residual = bn > 0 ? rn / bn : 0.0;
  // face gradients of the final p (xf is unchanged by this second pass)
  face_gradient(s, p, t, grad, xf);
  if (nf) {
    hipLaunchKernelGGL(k_corrected_flux, dim3(grid_for(nf)), dim3(kBlock), 0, s->stream, nf, owner,
                       neigh, active, Fs, coeff, p, xf, dt, flux);
    PPE_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(k_corrected_velocity, dim3(gc), dim3(kBlock), 0, s->stream, nc, aptr, anbr,
                     aface, active, grad, ustar, dt / rho, u);
  PPE_LAUNCH_CHECK();
  PPE_HIP(hipStreamSynchronize(s->stream));
  if (out) *out = st;
  return status;
}

}  // namespace ppe
