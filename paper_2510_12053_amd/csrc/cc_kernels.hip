// gfx950 kernels of the Coordinate Condensation sweep.
//
// Data layout (internal, colour-sorted order; see cc_kernels.h):
//   positions and gradients: float64 structure-of-arrays, component c of
//     vertex v at [c*n + v];
//   element store: per packed local block p (a <= b) an array of m blocks of
//     D*D values, [(p*m + e)*D*D + r*D + s];
//   block rows of the free-free Hessian: CSR over free vertices with the
//     diagonal block first in every row, [slot*D*D + r*D + s];
//   basis: CSR over free vertices, rows sorted by internal id, [q*D*D + ...].
//
// Every reduction is a fixed-order tree (no floating-point atomics), so runs
// are bit-reproducible.

#include <math.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "cc_device.h"

namespace cc {

// Element Hessian: H_e[a,b] = scale * V_e * sum_r w_r (Q_r beta_a)(Q_r beta_b)^T
// H selects the output blocks: 0 all of them, 1 the first half of the packed
// blocks, 2 the second half (the element's eigensystem is formed either way).
template <typename T, int D, int H>
__device__ __forceinline__ void elem_hess_body(const MeshView& mv, int e, const double* __restrict__ x,
                                               T mu, T lam, int model, T scale, T* __restrict__ out) {
  constexpr int K = D + 1, DD = D * D, NB = K * (K + 1) / 2;
  auto keep = [](int p) { return H == 0 || (H == 1 ? p < NB / 2 : p >= NB / 2); };
  if (e >= mv.m) return;
  T F[D][D], beta[K][D], vol;
  load_element<T, D>(mv, e, x, F, beta, vol);
  T acc[NB][DD];
#pragma unroll
  for (int p = 0; p < NB; ++p)
#pragma unroll
    for (int r = 0; r < DD; ++r) acc[p][r] = T(0);
  // y[a] = Q beta_a and z[a] = P beta_a (the vertex-a rows of the mode's
  // matrices); block (a, b) gains w y[a] z[b]^T
  auto rows = [&](const T (&M)[D][D], T (&y)[K][D]) {
#pragma unroll
    for (int a = 1; a < K; ++a)
#pragma unroll
      for (int r = 0; r < D; ++r) {
        T s = T(0);
#pragma unroll
        for (int q = 0; q < D; ++q) s += M[r][q] * beta[a][q];
        y[a][r] = s;
      }
#pragma unroll
    for (int r = 0; r < D; ++r) {
      T s = T(0);
#pragma unroll
      for (int a = 1; a < K; ++a) s += y[a][r];
      y[0][r] = -s;
    }
  };
  projected_eigs<T, D>(F, mu, lam, model, [&](T w, const T (&Q)[D][D], const T (&P)[D][D], bool same) {
    T y[K][D], z[K][D];
    rows(Q, y);
    if (same) {
#pragma unroll
      for (int a = 0; a < K; ++a)
#pragma unroll
        for (int r = 0; r < D; ++r) z[a][r] = y[a][r];
    } else {
      rows(P, z);
    }
#pragma unroll
    for (int a = 0; a < K; ++a) {
      T wy[D];
#pragma unroll
      for (int r = 0; r < D; ++r) wy[r] = w * y[a][r];
#pragma unroll
      for (int b = a; b < K; ++b)
        if (keep(pidx<K>(a, b)))
#pragma unroll
          for (int r = 0; r < D; ++r)
#pragma unroll
            for (int s = 0; s < D; ++s) acc[pidx<K>(a, b)][r * D + s] += wy[r] * z[b][s];
    }
  });
  const T f = scale * vol;
  const int m = mv.m;
#pragma unroll
  for (int p = 0; p < NB; ++p)
    if (keep(p))
#pragma unroll
      for (int r = 0; r < DD; ++r) out[((size_t)p * m + e) * DD + r] = f * acc[p][r];
}

// Element and assembly kernels run one thread per element / block slot in
// 64-thread workgroups: a few thousand elements then spread over most CUs
// instead of a few dozen (the per-element work is a long serial chain).
// In float64 the element kernel gives each workgroup of EWG elements two
// waves, each accumulating half of the output blocks: one wave holding all
// ten 3x3 float64 accumulators spills registers.
constexpr int EWG = 64;
template <typename T> constexpr int elem_threads() { return sizeof(T) == 8 ? 2 * EWG : EWG; }

// Element index of slot idx: idx itself, or entry idx of a list of ecount
// elements (past its end: m, which the body skips).
__device__ __forceinline__ int elem_of(const MeshView& mv, int idx, const int* elist, int ecount) {
  if (elist == nullptr) return idx;
  return idx < ecount ? elist[idx] : mv.m;
}

template <typename T, int D>
__device__ __forceinline__ void elem_hess_split(const MeshView& mv, int e0, const double* __restrict__ x,
                                                T mu, T lam, int model, T scale, T* __restrict__ out,
                                                const int* elist = nullptr, int ecount = 0) {
  if constexpr (sizeof(T) == 8) {
    const int e = elem_of(mv, e0 + threadIdx.x % EWG, elist, ecount);
    if (threadIdx.x < EWG) elem_hess_body<T, D, 1>(mv, e, x, mu, lam, model, scale, out);
    else elem_hess_body<T, D, 2>(mv, e, x, mu, lam, model, scale, out);
  } else {
    elem_hess_body<T, D, 0>(mv, elem_of(mv, e0 + threadIdx.x, elist, ecount), x, mu, lam, model, scale, out);
  }
}
constexpr int LS_WIDTH = 8;   // backtracking halvings evaluated per launch

template <typename T, int D, bool FCR>
__global__ void __launch_bounds__(elem_threads<T>()) k_elem_hess(MeshView mv, const double* __restrict__ x,
                                                                 T mu, T lam, int model, T scale,
                                                                 T* __restrict__ out, const int* elist,
                                                                 int ecount) {
  elem_hess_split<T, D>(mv, blockIdx.x * EWG, x, mu, lam, FCR ? model : MAT_SNH, scale, out, elist, ecount);
}

// R_j^T g_j (g itself without rotations), rounded to T once.
template <typename T, int D>
__device__ __forceinline__ void rotate_transpose(const double* rot, int j, const double (&gd)[D], T (&gj)[D]) {
  if (rot != nullptr) {
    const auto* Rj = gptr(rot) + (size_t)j * D * D;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      double acc = 0.0;
#pragma unroll
      for (int l = 0; l < D; ++l) acc += Rj[l * D + c] * gd[l];
      gj[c] = T(acc);
    }
  } else {
#pragma unroll
    for (int c = 0; c < D; ++c) gj[c] = T(gd[c]);
  }
}

// The band record of block slot t (row j) of a dense-basis mesh, when t is an
// upper slot: w R_j^T H_jk R_k, as a BandRec with the band position of k, or
// (mv.tile) as a tile record, whose diagonal block carries R_j^T g_j in its
// fourth row when g is given.
template <typename T, int D>
__device__ __forceinline__ void band_rec_write(const MeshView& mv, int t, int j, const T* blk, const double* g) {
  constexpr int DD = D * D;
  const bool tile = sizeof(T) == 4 && D == 3 && mv.tile;
  const int qp = tile ? mv.tb_slot[t] : mv.hq_slot[t];
  if (qp < 0) return;
  const int k = mv.colidx[t];
  const T w = k == j ? T(0.5) : T(1);
  T b[DD];
#pragma unroll
  for (int r = 0; r < DD; ++r) b[r] = w * blk[r];
  if (mv.rot != nullptr) {
    T Rj[DD], Rk[DD], tmp[DD];
#pragma unroll
    for (int r = 0; r < DD; ++r) {
      Rj[r] = T(mv.rot[(size_t)j * DD + r]);
      Rk[r] = T(mv.rot[(size_t)k * DD + r]);
    }
#pragma unroll
    for (int r = 0; r < D; ++r)               // tmp = B R_k
#pragma unroll
      for (int c = 0; c < D; ++c) {
        T acc = T(0);
#pragma unroll
        for (int l = 0; l < D; ++l) acc += b[r * D + l] * Rk[l * D + c];
        tmp[r * D + c] = acc;
      }
#pragma unroll
    for (int r = 0; r < D; ++r)               // b = R_j^T tmp
#pragma unroll
      for (int c = 0; c < D; ++c) {
        T acc = T(0);
#pragma unroll
        for (int l = 0; l < D; ++l) acc += Rj[l * D + r] * tmp[l * D + c];
        b[r * D + c] = acc;
      }
  }
  if constexpr (sizeof(T) == 4 && D == 3) {
    if (tile) {
      float gj[3] = {0.f, 0.f, 0.f};
      if (k == j && g != nullptr) {
        double gd[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) gd[c] = g[(size_t)c * mv.n + j];
        rotate_transpose<T, D>(mv.rot, j, gd, gj);
      }
      typedef float f4 __attribute__((ext_vector_type(4)));
      f4* rec = reinterpret_cast<f4*>(mv.tb) + (size_t)qp * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) rec[c] = f4{b[c], b[3 + c], b[6 + c], gj[c]};
      return;
    }
  }
  auto* rec = reinterpret_cast<BandRec<T, D>*>(mv.hq) + qp;
#pragma unroll
  for (int r = 0; r < DD; ++r) rec->h[r] = b[r];
  rec->pos = mv.bpos[k];
}

// Block rows: every slot sums its element contributions (fixed order), plus
// the mass on the diagonal.
template <typename T, int D>
__device__ __forceinline__ void assemble_body(const MeshView& mv, int tt, const T* __restrict__ est,
                                              T w_in, T* __restrict__ hb, const double* g,
                                              const int* slist = nullptr, int scount = 0) {
  constexpr int K = D + 1, DD = D * D;
  if (tt >= (slist ? scount : mv.nnzb)) return;
  // slots row by row in caller order of the rows: neighbouring threads then
  // read the blocks of neighbouring elements (a colour's list keeps that order)
  const int t = slist ? slist[tt] : (mv.aorder ? mv.aorder[tt] : tt);
  T acc[DD];
#pragma unroll
  for (int r = 0; r < DD; ++r) acc[r] = T(0);
  const int m = mv.m;
  // Contributions are summed in list order (so results are reproducible bit
  // for bit), with the blocks of four consecutive entries loaded before any
  // is added: a diagonal slot gathers one block per incident element, and a
  // chain of dependent index and block loads would set its time.
  const int c1 = mv.cptr[t + 1];
  int c = mv.cptr[t];
  for (; c + 4 <= c1; c += 4) {
    T v[4][DD];
    bool tr[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int pk = mv.centry[c + q];
      const int e = pk >> 4, a = (pk >> 2) & 3, b = pk & 3;
      tr[q] = a > b;
      const T* blk = est + ((size_t)pidx<K>(tr[q] ? b : a, tr[q] ? a : b) * m + e) * DD;
#pragma unroll
      for (int r = 0; r < DD; ++r) v[q][r] = blk[r];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < D; ++r)
#pragma unroll
        for (int s = 0; s < D; ++s) acc[r * D + s] += tr[q] ? v[q][s * D + r] : v[q][r * D + s];
  }
  for (; c < c1; ++c) {
    const int pk = mv.centry[c];
    const int e = pk >> 4, a = (pk >> 2) & 3, b = pk & 3;
    if (a <= b) {
      const T* blk = est + ((size_t)pidx<K>(a, b) * m + e) * DD;
#pragma unroll
      for (int r = 0; r < DD; ++r) acc[r] += blk[r];
    } else {
      const T* blk = est + ((size_t)pidx<K>(b, a) * m + e) * DD;
#pragma unroll
      for (int r = 0; r < D; ++r)
#pragma unroll
        for (int s = 0; s < D; ++s) acc[r * D + s] += blk[s * D + r];
    }
  }
  const int j = mv.blkrow[t];
  if (mv.colidx[t] == j) {
    const T mj = w_in * T(mv.mass[j]);
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r * D + r] += mj;
  }
#pragma unroll
  for (int r = 0; r < DD; ++r) hb[(size_t)t * DD + r] = acc[r];
  if (mv.hq != nullptr) band_rec_write<T, D>(mv, t, j, acc, g);
}

template <typename T, int D>
__global__ void __launch_bounds__(EWG) k_assemble(MeshView mv, const T* __restrict__ est, T w_in,
                                                  T* __restrict__ hb, const double* g, const int* slist,
                                                  int scount) {
  assemble_body<T, D>(mv, blockIdx.x * EWG + threadIdx.x, est, w_in, hb, g, slist, scount);
}

// Vertex of gradient slot idx: the free vertices in caller order, so that
// neighbouring lane groups walk overlapping element stars (nf: no vertex).
__device__ __forceinline__ int grad_vertex(const MeshView& mv, int idx) {
  if (idx >= mv.nf) return mv.nf;
  return mv.sorder ? mv.sorder[idx] : idx;
}

// Free-vertex gradient in float64: G lanes per vertex share its star.
// Returns g_j . g_j on the group's first lane, 0 elsewhere.
template <int D, int G, bool FCR>
__device__ __forceinline__ double gradient_body(const MeshView& mv, int j, int lane,
                                                const double* __restrict__ x,
                                                const double* __restrict__ xt, const Material& mat,
                                                double* __restrict__ g) {
  const int n = mv.n;
  double acc[D];
#pragma unroll
  for (int c = 0; c < D; ++c) acc[c] = 0.0;
  if (j < mv.nf) {
    for (int t = mv.star_ptr[j] + lane; t < mv.star_ptr[j + 1]; t += G) {
      const int pk = mv.star[t];
      const int e = pk >> 2, a = pk & 3;
      double F[D][D], beta[D + 1][D], vol, P[D][D];
      load_element<double, D>(mv, e, x, F, beta, vol);
      material_pk1<double, D>(F, mat.mu, mat.lam, FCR ? mat.model : MAT_SNH, P);
#pragma unroll
      for (int r = 0; r < D; ++r) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < D; ++q) s += P[r][q] * beta[a][q];
        acc[r] += vol * s;
      }
    }
  }
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1)
#pragma unroll
    for (int c = 0; c < D; ++c) acc[c] += __shfl_xor(acc[c], off, G);
  double gsq = 0.0;
  if (j < mv.nf && lane == 0) {
    const double mj = mv.mass[j];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      const double gj = mat.w_in * mj * (x[c * n + j] - xt[c * n + j]) +
                        mat.s_el * (acc[c] - mj * mat.grav[c]);
      g[c * n + j] = gj;
      gsq += gj * gj;
    }
  }
  return gsq;
}

template <int D, int G, bool FCR>
__global__ void __launch_bounds__(WG) k_gradient(MeshView mv, const double* __restrict__ x,
                                                 const double* __restrict__ xt, Material mat,
                                                 double* __restrict__ g,
                                                 double* __restrict__ partials) {
  __shared__ double red[WG];
  const double gsq = gradient_body<D, G, FCR>(mv, grad_vertex(mv, blockIdx.x * (WG / G) + threadIdx.x / G),
                                         threadIdx.x % G, x, xt, mat, g);
  const double tot = block_sum<WG>(gsq, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// Vertex of thread slot idx in [0, v1 - v0): a whole-mesh sweep visits the
// free vertices in caller order, so neighbouring slots share rows of H (the
// colour-sorted internal order scatters them over the mesh); a colour sweep
// takes its colour's range.
__device__ __forceinline__ int sweep_vertex(const MeshView& mv, int v0, int v1, int idx) {
  return (v0 == 0 && v1 == mv.nf && mv.sorder) ? mv.sorder[idx] : v0 + idx;
}

// Workgroups are dealt to the 8 XCDs in turn; renumber block b of nb so that
// the blocks one XCD runs cover a contiguous range (one L2 per XCD).
__device__ __forceinline__ int xcd_block(int b, int nb) {
  const int q = nb / 8, r = nb % 8, x = b % 8, k = b / 8;
  return x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

// Generic condensation kernel: G lanes per vertex, basis and support from
// global memory.  The support position of a neighbour comes from the slot map
// when the mesh has one, else from a binary search in the support row.
// With `stage` non-null (the same for the whole workgroup) each vertex group
// owns cap * D * D values of it: a support row of up to cap blocks is copied
// there with contiguous loads (and rotated once for a corotated basis), so the
// U_i[k] lookups of the slot-map path read LDS instead of scattered global
// blocks.
template <typename T, int D, int G>
__device__ __forceinline__ void prep_body(const MeshView& mv, int method, int i, bool active, int lane,
                                          const T* __restrict__ hb, T* __restrict__ KL,
                                          unsigned long long* __restrict__ fb,
                                          T* __restrict__ stage = nullptr, int cap = 0) {
  constexpr int DD = D * D;
  const T* Ub = basis_of<T>(mv);
  T A[DD], Ht[DD];
#pragma unroll
  for (int r = 0; r < DD; ++r) A[r] = Ht[r] = T(0);
  int64_t sp0 = 0, sp1 = 0;
  if (active && method != 0) supp_range(mv, i, sp0, sp1);
  const T* Us = nullptr;   // staged, rotated support row of vertex i
  if (stage) {
    const bool st = active && method != 0 && mv.smap && sp1 - sp0 <= cap;
    T* my = stage + (size_t)(threadIdx.x / G) * cap * DD;
    if (st)
      for (int e = lane; e < (int)(sp1 - sp0) * DD; e += G) my[e] = Ub[sp0 * DD + e];
    __syncthreads();
    if (mv.rot) {
      if (st)
        for (int q = lane; q < (int)(sp1 - sp0); q += G) {
          T b[DD];
#pragma unroll
          for (int r = 0; r < DD; ++r) b[r] = my[q * DD + r];
          rotate_block<T, D>(mv.rot, mv.sidx[sp0 + q], b);
#pragma unroll
          for (int r = 0; r < DD; ++r) my[q * DD + r] = b[r];
        }
      __syncthreads();
    }
    if (st) Us = my;
  }
  if (active && method != 0 && mv.smap) {
    // Sparse support with a slot map: the blocks (j, k), k >= j, of row j
    // whose column lies in supp(i) come with k's support position, so the
    // loads of H_jk and U_i[k] do not wait on a search.  H is symmetric, so
    // with W = sum_{k > j} H_jk U_i[k] + 1/2 H_jj U_i[j] and
    // Y = sum_j U_i[j]^T W, Ht = Y + Y^T (formed after the lane reduction).
    const int nw = mv.smap_words;
    for (int64_t q = sp0 + lane; q < sp1; q += G) {
      const int a = (int)(q - sp0);
      const uint32_t* sm = mv.smap + (size_t)q * (nw + 1);
      const int t0 = (int)sm[0];
      T Uj[DD], W[DD];
      if (Us) {
#pragma unroll
        for (int r = 0; r < DD; ++r) Uj[r] = Us[(q - sp0) * DD + r];
      } else {
#pragma unroll
        for (int r = 0; r < DD; ++r) Uj[r] = Ub[q * DD + r];
        if (mv.rot) rotate_block<T, D>(mv.rot, mv.sidx[q], Uj);
      }
#pragma unroll
      for (int r = 0; r < DD; ++r) W[r] = T(0);
      for (int w = 0; w < nw; ++w) {
        const uint32_t word = sm[1 + w];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int code = (word >> (8 * b)) & 255;
          if (code == SMAP_SKIP) continue;
          const T* H = hb + (size_t)(t0 + 4 * w + b) * DD;
          T Hl[DD];
#pragma unroll
          for (int r = 0; r < DD; ++r) Hl[r] = H[r];
          if (code == SMAP_SELF) {            // block (j, i): A += H_ji^T U_i[j]
#pragma unroll
            for (int r = 0; r < D; ++r)
#pragma unroll
              for (int c = 0; c < D; ++c) {
                T acc = T(0);
#pragma unroll
                for (int l = 0; l < D; ++l) acc += Hl[l * D + r] * Uj[l * D + c];
                A[r * D + c] += acc;
              }
            continue;
          }
          T Uk[DD];
          if (Us) {
#pragma unroll
            for (int r = 0; r < DD; ++r) Uk[r] = Us[code * DD + r];
          } else {
            const int64_t qk = sp0 + code;
#pragma unroll
            for (int r = 0; r < DD; ++r) Uk[r] = Ub[qk * DD + r];
            if (mv.rot) rotate_block<T, D>(mv.rot, mv.sidx[qk], Uk);
          }
          if (code == a)                      // diagonal block: half weight (exact)
#pragma unroll
            for (int r = 0; r < DD; ++r) Uk[r] *= T(0.5);
#pragma unroll
          for (int r = 0; r < D; ++r)         // W += H_jk U_i[k]
#pragma unroll
            for (int c = 0; c < D; ++c) {
              T acc = W[r * D + c];
#pragma unroll
              for (int l = 0; l < D; ++l) acc += Hl[r * D + l] * Uk[l * D + c];
              W[r * D + c] = acc;
            }
        }
      }
#pragma unroll
      for (int r = 0; r < D; ++r)             // Y += U_i[j]^T W
#pragma unroll
        for (int c = 0; c < D; ++c) {
          T acc = T(0);
#pragma unroll
          for (int l = 0; l < D; ++l) acc += Uj[l * D + r] * W[l * D + c];
          Ht[r * D + c] += acc;
        }
    }
  } else if (active && method != 0) {
    for (int64_t q = sp0 + lane; q < sp1; q += G) {
      const int j = supp_vertex(mv, q, sp0);
      if (j == i) continue;                   // the zero own block of a dense row
      T Uj[DD];
#pragma unroll
      for (int r = 0; r < DD; ++r) Uj[r] = Ub[q * DD + r];
      if (mv.rot) rotate_block<T, D>(mv.rot, j, Uj);
      accum_row<T, D>(mv, i, j, Uj, hb, [&](int k, T* Uk) -> bool {
        const int64_t qk = find_slot(mv, sp0, sp1, i, k);
        if (qk < 0) return false;
#pragma unroll
        for (int r = 0; r < DD; ++r) Uk[r] = Ub[(size_t)qk * DD + r];
        if (mv.rot) rotate_block<T, D>(mv.rot, k, Uk);
        return true;
      }, A, Ht);
    }
  }
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1)
#pragma unroll
    for (int r = 0; r < DD; ++r) {
      A[r] += __shfl_xor(A[r], off, G);
      Ht[r] += __shfl_xor(Ht[r], off, G);
    }
  if (!active || lane != 0) return;
  if (mv.smap) {                              // Ht = Y + Y^T
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
      for (int c = r; c < D; ++c) {
        const T y = Ht[r * D + c] + Ht[c * D + r];
        Ht[r * D + c] = y;
        Ht[c * D + r] = y;
      }
  }
  cc_finish<T, D>(mv, method, i, sp1 == sp0, A, Ht, hb, KL, fb);
}

template <typename T, int D, int G>
__global__ void __launch_bounds__(WG) k_cc_prep(MeshView mv, int method, int v0, int v1,
                                                const T* __restrict__ hb, T* __restrict__ KL,
                                                unsigned long long* __restrict__ fb, int cap) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int idx = xcd_block(blockIdx.x, gridDim.x) * (WG / G) + threadIdx.x / G;
  const bool act = idx < v1 - v0;
  prep_body<T, D, G>(mv, method, act ? sweep_vertex(mv, v0, v1, idx) : v0, act, threadIdx.x % G, hb, KL,
                     fb, cap > 0 ? reinterpret_cast<T*>(smem_raw) : nullptr, cap);
}

// Exact-basis condensation of TV vertices per workgroup (Method, Eqs. block
// and schur: A_i = H_iC U_i, Ht_i = U_i^T H_CC U_i, b_i = U_i^T g_C; with
// corotation every U_i[j] is R_j U_i[j], Eq. rotation).
//
// The basis rows are stored in band order (MeshView::bvert), in which every
// block (j, k) of H with k after j has k within band_w positions of j.  H is
// symmetric, so with X_jk = U_j^T H''_jk U_k, H''_jk = R_j^T H_jk R_k,
//   Ht = sum_{j,k} X_jk = Y + Y^T,  Y = sum_j U_j^T W_j,
//   W_j = sum_{k >= j} w_jk H''_jk U_k  (w = 1/2 on the diagonal block),
// and only the upper blocks are read, from the BandRec list hq (rotated and
// weighted there once per Hessian, not once per basis row).  The workgroup
// walks the band in chunks of CH positions, one thread per row j of the
// chunk; row j needs U at positions [j, j + band_w], so the TV rows live in
// an LDS ring of R >= CH + band_w positions, refilled one chunk ahead: the
// global loads of chunk c + 1's new positions are issued before chunk c's
// products and stored after them.  A ring slot holds the TV blocks of one
// position contiguously, padded to an odd number of words, so a block read
// is one address and constant offsets, and the threads of a wave, which
// take consecutive positions (whose columns are, on structured grids,
// consecutive too), hit distinct banks.  Every H block serves the TV rows of
// the workgroup from registers.
// A_i = sum_k H_ik R_k U_i[k] comes from row i in global memory (one wave
// per vertex; the row was just streamed through L2).
//
// With g given (Jacobi sweeps), b_i = U_i^T (R^T g)_C is also accumulated
// from the staged rows and stored in bout (component-major, stride n); the
// finish kernel then writes the direction itself.
template <typename T, int D>
__device__ __forceinline__ void band_load(const MeshView& mv, const T* __restrict__ Ub, int row, int pos,
                                          T (&blk)[D * D]) {
  constexpr int DD = D * D;
  const auto* src = gptr(Ub) + ((size_t)row * mv.nf + pos) * DD;
#pragma unroll
  for (int r = 0; r < DD; ++r) blk[r] = src[r];
}

// Raw buffer resource over `bytes` bytes at p (offsets past the end read
// as zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// A BandRec as raw dwords, loaded 16 bytes at a time from byte offset off.
template <typename T, int D>
struct RecWords {
  static constexpr int N = sizeof(BandRec<T, D>) / 4;
  uint32_t w[N];
  __device__ __forceinline__ void fetch(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
#pragma unroll
    for (int c = 0; c < N / 4; ++c) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16u * c, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * c + e] = v[e];
    }
  }
  __device__ __forceinline__ T h(int r) const {
    if constexpr (sizeof(T) == 4) {
      return __builtin_bit_cast(float, w[r]);
    } else {
      return __builtin_bit_cast(double, (uint64_t)w[2 * r] | ((uint64_t)w[2 * r + 1] << 32));
    }
  }
  __device__ __forceinline__ int pos() const { return (int)w[D * D * sizeof(T) / 4]; }
};

// Sum over the 64 lanes of a wave, valid in lane 63: rotations within each
// row of 16 lanes leave the row sum in every lane of the row, then two row
// broadcasts add rows 0-1 into row 3 (DPP, no LDS traffic).
__device__ __forceinline__ float dpp_step(float x, int y) { return x + __builtin_bit_cast(float, y); }
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROWS, 0xf, false);
  return dpp_step(x, y);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
  return x + __builtin_bit_cast(double, (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32));
}
template <typename T>
__device__ __forceinline__ T wave_sum63(T x) {
  x = dpp_add<0x128, 0xf>(x);   // row_ror:8
  x = dpp_add<0x124, 0xf>(x);   // row_ror:4
  x = dpp_add<0x122, 0xf>(x);   // row_ror:2
  x = dpp_add<0x121, 0xf>(x);   // row_ror:1
  x = dpp_add<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
  x = dpp_add<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
  return x;
}

template <int W> struct UnitVec;
template <> struct UnitVec<1> { typedef uint32_t type; };
template <> struct UnitVec<2> { typedef uint32_t type __attribute__((ext_vector_type(2))); };
template <> struct UnitVec<4> { typedef uint32_t type __attribute__((ext_vector_type(4))); };

// The TV blocks of one ring slot in registers, read and written one access
// unit at a time (ring_slot_unit).
template <typename T, int D, int TV>
struct SlotRegs {
  static constexpr int UW = ring_slot_unit(TV, D, (int)sizeof(T)) / 4;   // words per unit
  static constexpr int NW = (TV * D * D * (int)sizeof(T) / 4 + UW - 1) / UW * UW;   // data words, whole units
  typedef typename UnitVec<UW>::type unit_t;
  uint32_t w[NW];
  __device__ __forceinline__ void load(const uint32_t* slot) {
    const unit_t* src = reinterpret_cast<const unit_t*>(slot);
#pragma unroll
    for (int c = 0; c < NW / UW; ++c) {
      const unit_t u = src[c];
      if constexpr (UW == 1) {
        w[c] = u;
      } else {
#pragma unroll
        for (int e = 0; e < UW; ++e) w[c * UW + e] = u[e];
      }
    }
  }
  __device__ __forceinline__ void store(uint32_t* slot) const {
    unit_t* dst = reinterpret_cast<unit_t*>(slot);
#pragma unroll
    for (int c = 0; c < NW / UW; ++c) {
      unit_t u;
      if constexpr (UW == 1) {
        u = w[c];
      } else {
#pragma unroll
        for (int e = 0; e < UW; ++e) u[e] = w[c * UW + e];
      }
      dst[c] = u;
    }
  }
  __device__ __forceinline__ T get(int idx) const {        // idx = v * D*D + r
    if constexpr (sizeof(T) == 4) {
      return __builtin_bit_cast(float, w[idx]);
    } else {
      return __builtin_bit_cast(double, (uint64_t)w[2 * idx] | ((uint64_t)w[2 * idx + 1] << 32));
    }
  }
  __device__ __forceinline__ void set(int idx, T x) {
    if constexpr (sizeof(T) == 4) {
      w[idx] = __builtin_bit_cast(uint32_t, x);
    } else {
      const uint64_t b = __builtin_bit_cast(uint64_t, x);
      w[2 * idx] = (uint32_t)b;
      w[2 * idx + 1] = (uint32_t)(b >> 32);
    }
  }
};

// Segment seg's (1 .. nseg - 1) sums of vertex i: its part of Ht and of b.
// Segment 0 leaves its own in the K, L slots and the direction.
template <typename T, int D>
__device__ __forceinline__ T* seg_sums(const MeshView& mv, int seg, int i) {
  return reinterpret_cast<T*>(mv.segsum) + ((size_t)(seg - 1) * mv.nf + i) * (D * D + D);
}

// The end of the band kernel's workgroup: per vertex, A_i from its basis row in
// global memory (one wave per vertex) into its K slot, and Ht_i = Y + Y^T and b_i
// from the workgroup's sums tot ([vertex][Y, then b]).
template <typename T, int D>
__device__ __forceinline__ void band_tail(const MeshView& mv, int i0, int nv, int w, int nw,
                                          const T* __restrict__ hb, T* __restrict__ KL, const T* tot,
                                          double* __restrict__ bout) {
  constexpr int DD = D * D, NR = DD + D;
  const T* Ub = basis_of<T>(mv);
  const int l = threadIdx.x % 64;
  // one wave per row (rows w, w + nw, ... when the chunk has fewer waves
  // than rows)
  for (int v = w; v < nv; v += nw) {
    const int i = i0 + v;
    T A[DD];
#pragma unroll
    for (int r = 0; r < DD; ++r) A[r] = T(0);
    const int q1 = gptr(mv.rowptr)[i + 1];
    for (int q = gptr(mv.rowptr)[i] + 1 + l; q < q1; q += 64) {
      const int k = gptr(mv.colidx)[q];
      T Uk[DD];
      band_load<T, D>(mv, Ub, i, gptr(mv.bpos)[k], Uk);
      if (mv.rot != nullptr) rotate_block<T, D>(mv.rot, k, Uk);
      const auto* H = gptr(hb) + (size_t)q * DD;
#pragma unroll
      for (int r = 0; r < D; ++r)
#pragma unroll
        for (int c = 0; c < D; ++c) {
          T acc = T(0);
#pragma unroll
          for (int t = 0; t < D; ++t) acc += H[r * D + t] * Uk[t * D + c];
          A[r * D + c] += acc;
        }
    }
#pragma unroll
    for (int r = 0; r < DD; ++r) A[r] = wave_sum63(A[r]);
    if (l != 63) continue;
    // A and Ht go to the vertex's K, L slots; dm_finish_body turns them into
    // K and L with one thread per vertex.  b_i = U_i^T (R^T g)_C, the
    // corotated basis's U_i^T g_C.
    const T* Yt = tot + v * NR;
    auto* out = gptr_w(KL) + (size_t)i * 2 * DD;
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c) {
        out[r * D + c] = A[r * D + c];
        out[DD + r * D + c] = Yt[r * D + c] + Yt[c * D + r];
      }
    if (bout != nullptr)
#pragma unroll
      for (int r = 0; r < D; ++r) gptr_w(bout)[(size_t)r * mv.n + i] = double(Yt[DD + r]);
  }
}


template <typename T, int D, int TV, int CH>
__device__ __forceinline__ void prep_band_body(const MeshView& mv, int i0, int nv,
                                               const T* __restrict__ hb, T* __restrict__ KL, T* smem,
                                               const double* __restrict__ g, double* __restrict__ bout, int seg,
                                               int nseg) {
  constexpr int DD = D * D, NW = CH / 64, NR = DD + D, SLW = ring_slot_words(TV, D, sizeof(T));
  const int nf = mv.nf, n = mv.n, bw = mv.band_w;
  const int R = min(nf, CH + bw);                   // ring length (band_ring)
  // position pos >= p0 (the current chunk's start) lives in slot
  // (pos - p0 + p0's slot) mod R; pos - p0 < CH + bw, so one conditional
  // subtraction of R reduces it
  auto wrap = [&](int t) { return (int)min((unsigned)t, (unsigned)(t - R)); };
  uint32_t* ring = reinterpret_cast<uint32_t*>(smem);              // [R][SLW] words
  T* red = reinterpret_cast<T*>(ring + (size_t)R * SLW);          // [NW][TV][NR]
  const T* Ub = basis_of<T>(mv);
  constexpr uint32_t RB = sizeof(BandRec<T, D>);
  const __amdgpu_buffer_rsrc_t hrs = buf_rsrc(mv.hq, (uint32_t)((size_t)mv.qmax * nf * RB));
  const int tid = threadIdx.x;
  int rows[TV];
#pragma unroll
  for (int v = 0; v < TV; ++v) rows[v] = i0 + (v < nv ? v : 0);
  auto put = [&](int pos, T (&blk)[TV][DD]) {
    SlotRegs<T, D, TV> sr;
#pragma unroll
    for (int v = 0; v < TV; ++v)
#pragma unroll
      for (int r = 0; r < DD; ++r) sr.set(v * DD + r, blk[v][r]);
    sr.store(ring + (size_t)pos * SLW);            // pos: a slot
  };
  // one buffer resource per basis row (a dense basis can pass 4 GiB, one
  // row cannot), so a block's offset is pos * D*D * sizeof(T)
  __amdgpu_buffer_rsrc_t urs[TV];
#pragma unroll
  for (int v = 0; v < TV; ++v)
    urs[v] = buf_rsrc(Ub + (size_t)rows[v] * nf * DD, (uint32_t)((size_t)nf * DD * sizeof(T)));
  auto fetch = [&](int pos, T (&blk)[TV][DD]) {
    const uint32_t off = (uint32_t)pos * (uint32_t)(DD * sizeof(T));
#pragma unroll
    for (int v = 0; v < TV; ++v)
#pragma unroll
      for (int r = 0; r < DD; ++r) {
        if constexpr (sizeof(T) == 4) {
          blk[v][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(urs[v], off + 4u * r, 0, 0));
        } else {
          const auto u = __builtin_amdgcn_raw_buffer_load_b64(urs[v], off + 8u * r, 0, 0);
          blk[v][r] = __builtin_bit_cast(double, u);
        }
      }
  };
  // band rows [pa, pb): whole chunks, the segment's share of them
  const int nch = (nf + CH - 1) / CH, pa = nch * seg / nseg * CH, pb = min(nf, nch * (seg + 1) / nseg * CH);
  int lo = min(nf, pa + R);                         // first fill: positions [pa, lo) in slots [0, lo - pa)
  for (int pos = pa + tid; pos < lo; pos += CH) {
    T blk[TV][DD];
    fetch(pos, blk);
    put(pos - pa, blk);
  }
  int lo_slot = 0;                                  // slot of position lo
  int p0_slot = 0;                                  // slot of position p0
  __syncthreads();
  T Y[TV][DD], Bv[TV][D];
#pragma unroll
  for (int v = 0; v < TV; ++v) {
#pragma unroll
    for (int r = 0; r < DD; ++r) Y[v][r] = T(0);
#pragma unroll
    for (int r = 0; r < D; ++r) Bv[v][r] = T(0);
  }
  for (int p0 = pa; p0 < pb; p0 += CH) {
    // chunk p0 + CH needs positions up to p0 + 2 CH + bw: prefetch them
    const int nhi = min(nf, min(p0 + 2 * CH, pb) + bw);
    const int ppos = lo + tid;
    const bool pf = ppos < nhi;
    T pre[TV][DD];
    if (pf) fetch(ppos, pre);
    const int p = p0 + tid;
    const int cshift = p0_slot - p0;                // slot = wrap(pos + cshift)
    if (p < nf) {
      const int cnt = gptr(mv.bq_cnt)[p];
      T W[TV][DD];
      // W_j = sum_q H''_{j,q} U_{k(q)}.  Record 0 is the diagonal block
      // (always present), applied with the row's own U_j, which the Y update
      // below needs anyway, so that it costs no ring read of its own.  With
      // three or four float32 rows U_j is read first and the diagonal product
      // sets W (no clearing of the accumulators, which the compiler emits
      // twice around the loop's guard; three rows then hold two waves per
      // SIMD instead of three, which their LDS ring allows anyway on meshes
      // whose band is too wide for four); with fewer rows, whose occupancy
      // the extra live registers would cut, W is cleared and the diagonal
      // block comes last.  The other upper blocks run in a software pipeline unrolled by
      // two: block q + 1 (its H and column) is loaded while block q's LDS
      // reads and products run.  Records past the row's count are zero
      // padding or past the end of the buffer (read as zero) and are never
      // used.
      constexpr bool own_first = sizeof(T) == 4 && TV >= 3;
      auto product = [&](const RecWords<T, D>& rc, const SlotRegs<T, D, TV>& sr, bool first) {
#pragma unroll
        for (int v = 0; v < TV; ++v) {
          T U[DD];
#pragma unroll
          for (int r = 0; r < DD; ++r) U[r] = sr.get(v * DD + r);
#pragma unroll
          for (int r = 0; r < D; ++r)
#pragma unroll
            for (int c = 0; c < D; ++c) {
              T acc = first ? rc.h(r * D) * U[c] : W[v][r * D + c] + rc.h(r * D) * U[c];
#pragma unroll
              for (int l = 1; l < D; ++l) acc += rc.h(r * D + l) * U[l * D + c];
              W[v][r * D + c] = acc;
            }
        }
      };
      auto consume = [&](const RecWords<T, D>& rc) {
        SlotRegs<T, D, TV> sr;
        sr.load(ring + (size_t)wrap(rc.pos() + cshift) * SLW);
        product(rc, sr, false);
      };
      const uint32_t step = (uint32_t)nf * RB;
      uint32_t off = (uint32_t)p * RB;
      RecWords<T, D> rd, ra, rb;
      SlotRegs<T, D, TV> sj;
      rd.fetch(hrs, off);                           // the diagonal block
      off += step;
      ra.fetch(hrs, off);
      if constexpr (own_first) {
        sj.load(ring + (size_t)wrap(p + cshift) * SLW);
        product(rd, sj, true);
      } else {
#pragma unroll
        for (int v = 0; v < TV; ++v)
#pragma unroll
          for (int r = 0; r < DD; ++r) W[v][r] = T(0);
      }
      int q = 1;
      for (; q + 1 < cnt; q += 2) {
        rb.fetch(hrs, off + step);
        consume(ra);
        ra.fetch(hrs, off + 2 * step);
        consume(rb);
        off += 2 * step;
      }
      if (q < cnt) consume(ra);
      T gj[D];
      if (g != nullptr) {
        const int j = gptr(mv.bvert)[p];
        double gd[D];
#pragma unroll
        for (int c = 0; c < D; ++c) gd[c] = gptr(g)[(size_t)c * n + j];
        rotate_transpose<T, D>(mv.rot, j, gd, gj);
      }
      if constexpr (!own_first) {
        sj.load(ring + (size_t)wrap(p + cshift) * SLW);
        product(rd, sj, false);
      }
#pragma unroll
      for (int v = 0; v < TV; ++v) {
        T Uj[DD];
#pragma unroll
        for (int r = 0; r < DD; ++r) Uj[r] = sj.get(v * DD + r);
#pragma unroll
        for (int l = 0; l < D; ++l)
#pragma unroll
          for (int r = 0; r < D; ++r)
#pragma unroll
            for (int c = 0; c < D; ++c) Y[v][r * D + c] += Uj[l * D + r] * W[v][l * D + c];
        if (g != nullptr)
#pragma unroll
          for (int r = 0; r < D; ++r) {
            T acc = T(0);
#pragma unroll
            for (int l = 0; l < D; ++l) acc += Uj[l * D + r] * gj[l];
            Bv[v][r] += acc;
          }
      }
    }
    __syncthreads();                                // chunk p0's ring reads are done
    if (pf) put(wrap(lo_slot + tid), pre);
    if (nhi > lo) {
      lo_slot = wrap(lo_slot + (nhi - lo));
      lo = nhi;
    }
    p0_slot = wrap(p0_slot + CH);
    __syncthreads();
  }
#pragma unroll
  for (int v = 0; v < TV; ++v) {
#pragma unroll
    for (int r = 0; r < DD; ++r) Y[v][r] = wave_sum63(Y[v][r]);
#pragma unroll
    for (int r = 0; r < D; ++r) Bv[v][r] = wave_sum63(Bv[v][r]);
  }
  const int w = tid / 64, l = tid % 64;
  if (l == 63)
#pragma unroll
    for (int v = 0; v < TV; ++v) {
#pragma unroll
      for (int r = 0; r < DD; ++r) red[(w * TV + v) * NR + r] = Y[v][r];
#pragma unroll
      for (int r = 0; r < D; ++r) red[(w * TV + v) * NR + DD + r] = Bv[v][r];
    }
  __syncthreads();
  T* tot = smem;                                    // the ring is free now: [TV][NR]
  if (tid < TV * NR) {
    T acc = T(0);
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) acc += red[ww * TV * NR + tid];
    tot[tid] = acc;
  }
  __syncthreads();
  if (seg == 0) {
    band_tail<T, D>(mv, i0, nv, w, NW, hb, KL, tot, bout);
  } else if (tid < nv * NR) {
    const int v = tid / NR, k = tid % NR;
    const T* Yt = tot + v * NR;
    seg_sums<T, D>(mv, seg, i0 + v)[k] = k < DD ? Yt[k] + Yt[k % D * D + k / D] : Yt[k];
  }
}

// A_i = sum_k H_ik R_k U_i[k] of a tile workgroup's vertices, into their K slots
// (dm_finish_body reads them): 16 lanes per vertex, four vertices per wave.
template <int V>
__device__ __forceinline__ void tile_rows(const MeshView& mv, int i0, int nv, int w, const float* __restrict__ hb,
                                          float* __restrict__ KL) {
  if (w >= (V + 3) / 4) return;
  const int l = threadIdx.x % 64, v = w * 4 + l / 16, i = i0 + min(v, nv - 1);
  float A[9];
#pragma unroll
  for (int r = 0; r < 9; ++r) A[r] = 0.f;
  const int q1 = gptr(mv.rowptr)[i + 1];
  for (int q = gptr(mv.rowptr)[i] + 1 + l % 16; q < q1; q += 16) {
    const int k = gptr(mv.colidx)[q];
    float Uk[9];
    band_load<float, 3>(mv, mv.U_f, i, gptr(mv.bpos)[k], Uk);
    if (mv.rot != nullptr) rotate_block<float, 3>(mv.rot, k, Uk);
    const auto* H = gptr(hb) + (size_t)q * 9;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        float acc = 0.f;
#pragma unroll
        for (int t = 0; t < 3; ++t) acc += H[r * 3 + t] * Uk[t * 3 + c];
        A[r * 3 + c] += acc;
      }
  }
#pragma unroll
  for (int r = 0; r < 9; ++r) {                      // sums over the 16 lanes
    A[r] = dpp_add<0x128, 0xf>(A[r]);
    A[r] = dpp_add<0x124, 0xf>(A[r]);
    A[r] = dpp_add<0x122, 0xf>(A[r]);
    A[r] = dpp_add<0x121, 0xf>(A[r]);
  }
  if (l % 16 != 0 || v >= nv) return;
#pragma unroll
  for (int r = 0; r < 9; ++r) gptr_w(KL)[(size_t)i * 18 + r] = A[r];
}

// Exact-basis condensation of float32 3D meshes on the matrix cores: the sums
// of prep_band_body (W_j = sum_k w_jk H''_jk U_k over the upper blocks of row
// j, Y = sum_j U_j^T W_j, b = sum_j U_j^T R_j^T g_j) for 5 NG vertices per
// workgroup, CH positions of the band at a time.
//
// One v_mfma_f32_4x4x1 holds 16 independent 4 x 4 products.  The wave's four
// rows of 16 lanes take four band rows j; the 15 columns of five vertices'
// basis blocks are the lanes of a row (lane 15 idles), so that one
// instruction forms one column s of one block: W_j[., col] += H''_jk[., s]
// U_k[s, col].  The H'' column (four values: the block's three rows and, for
// the diagonal block, g_j[s], which accumulates b in the fourth) is broadcast
// to the row's four 4-lane blocks by the instruction itself (cbsz = 2), so a
// wave reads a block as 12 floats per band row straight from the tile records.
// Each product is a float32 FMA, as in prep_band_body; with three of four
// rows and 15 of 16 columns used it does 180 FMAs in 8 cycles against the
// 128 of two VALU instructions.  The U_j^T W_j products of the four band rows
// are one v_mfma_f32_16x16x4 per component: lane row = k, so U and W are its
// operands as they lie, and the vertices' 3 x 3 blocks lie on its diagonal.
//
// Position p of the basis rows lives in ring slot p mod R of its vertex, nine
// words as in memory, so a chunk's refill is a flat copy and the records'
// columns are LDS offsets computed once per mesh (tb_off), broadcast to a lane
// row by a DPP addition.  The lane rows' band rows are 16 positions apart: with
// nine words a slot and vertex strides of 3 mod 16 words, the 30 reads of a
// half wave hit 30 banks wherever the columns keep the rows' distance, as
// inside structured grids.  Rows past the last band row and blocks past a
// row's count are zero records on a valid slot.
//
// What bounds it: the issue of the 27 matrix instructions (288 cycles) and
// about 18 VALU ones (72) a wave spends on four band rows of five vertices; on
// the 41x11x11 bar these are two thirds of the busy cycles, the LDS is busy
// for half of them.  Two accumulator chains, since a dependent 4x4x1 product
// waits longer than its 8 cycles (a phase of the loop alone: 402 against 467
// cycles of 2.4 GHz).  The partial sums of a chunk are added up apart, which
// keeps the rounding of the sums over up to 35,000 positions at that of
// prep_band_body's many short ones.  Corotated, active launches against
// prep_band_body's: 41x11x11 bar 329 against 445 us (357 with its rows split),
// the 64-bar batch 2.99 against 3.13 ms on average, the 81x21x21 beam 17.9
// against 23.2 ms (in sixteen waves: one workgroup per CU fits, and with eight a
// step took 117 ms against 91).  Where it is not the better one: tile_fills,
// band_better.
template <int NG, int NS, int CH>
__device__ __forceinline__ void prep_tile_body(const MeshView& mv, int i0, int nv, const float* __restrict__ hb,
                                               float* __restrict__ KL, float* smem, double* __restrict__ bout,
                                               int seg, int nseg) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) float lds_float;
  constexpr int V = 5 * NG, NT = 64 * NS, SEG = CH / (4 * NS), NR = 12, PHASES = SEG * NG;
  constexpr int CFG = CH == TILE_CH[0] ? 0 : CH == TILE_CH[1] ? 1 : 2;
  constexpr uint32_t PB = TILE_Q * 48, OB = TILE_Q * 4;   // bytes of one band row's records and offsets
  static_assert(CH == TILE_CH[CFG] && NG == TILE_G[CFG] && NS == TILE_WAVES[CFG] && SEG * 4 * NS == CH &&
                    PHASES % 2 == 0 && TILE_Q == 8, "configuration");
  const int nf = mv.nf, nf9 = nf * 9;
  const int R = CFG == 0 ? TILE_RING : tile_ring(CFG + 1, nf, mv.band_w), VS = tile_stride(R);
  // band rows [pa, pb): the segment's share of the row in whole rings, so that
  // position p keeps its slot p mod R
  const int pa = tile_segment(nf, R, seg, nseg), pb = min(nf, tile_segment(nf, R, seg + 1, nseg));
  const int tid = threadIdx.x, l = tid % 64, w = __builtin_amdgcn_readfirstlane(tid / 64);
  // A vertex's row is copied into its ring in pieces of 64 words, one word per
  // lane.  What a piece reads past the row's end (the next row, or the
  // DENSE_F32_PAD words past the last) is never used.  The descriptor does not
  // check it: a piece's place is a scalar offset, which is not part of the check.
  static_assert(TILE_PIECE == 64, "one word per lane");
  constexpr int UC = CH * 9 / 64, NP = (V * UC + NS - 1) / NS;   // pieces of a chunk per vertex, per wave
  const __amdgpu_buffer_rsrc_t urs = buf_rsrc(mv.U_f + (size_t)i0 * nf9, (uint32_t)(nv * nf9 + DENSE_F32_PAD) * 4u);
  const uint32_t gl4 = (uint32_t)l * 4u;
  uint32_t wl4 = (uint32_t)(uintptr_t)(lds_float*)smem + gl4;
  asm volatile("" : "+v"(wl4));
  auto load_piece = [&](uint32_t at) { return __builtin_amdgcn_raw_buffer_load_b32(urs, gl4, at, 0); };
  auto put_piece = [&](uint32_t at, uint32_t x) {
    *(__attribute__((address_space(3))) uint32_t*)(uintptr_t)(wl4 + at) = x;
  };
  auto row4 = [&](int v) { return (uint32_t)((v < nv ? v : 0) * nf9) * 4u; };
  auto ring4 = [&](int v) { return (uint32_t)(v * VS) * 4u; };
  const int UF = R * 9 / 64, fill = V * UF;          // first fill: positions [pa, min(pa + R, nf))
  constexpr int FB = 17;                             // pieces in flight per wave
  uint32_t first[FB];
  auto fill_load = [&](int x0) {
#pragma unroll
    for (int e = 0; e < FB; ++e) {
      const int k = min(x0 + e * NS, fill - 1);
      first[e] = load_piece(row4(k / UF) + tile_fill_piece(pa, k % UF, nf) * 4u);
    }
  };
  fill_load(w);
  if (seg == 0) tile_rows<V>(mv, i0, nv, w, hb, KL); // A_i, while the fill is on its way
  for (int x0 = w; x0 < fill; x0 += FB * NS) {
#pragma unroll
    for (int e = 0; e < FB; ++e) {
      const int k = min(x0 + e * NS, fill - 1);
      put_piece(ring4(k / UF) + (uint32_t)(k % UF) * 256u, first[e]);
    }
    if (x0 + FB * NS < fill) fill_load(x0 + FB * NS);
  }
  // the wave's pieces of a chunk: bytes from the chunk's first position in the rows and in the ring
  uint32_t gat[NP], lat[NP];
#pragma unroll
  for (int e = 0; e < NP; ++e) {
    const int x = min(w + e * NS, V * UC - 1);
    gat[e] = row4(x / UC) + tile_piece(0, x % UC) * 4u;
    lat[e] = ring4(x / UC) + (uint32_t)(x % UC) * 256u;
    asm volatile("" : "+s"(gat[e]), "+s"(lat[e]));
  }
  const int q = l / 16, l16 = l % 16, col = min(l16, 14);
  // LDS byte address of the lane's column in ring slot 0 (opaque, so that a
  // read's address is one addition for every group)
  uint32_t lbase = (uint32_t)(uintptr_t)(lds_float*)(smem + col / 3 * VS + col % 3);
  asm volatile("" : "+v"(lbase));
  // the lane row's first band row of a chunk: the lane rows are SP = 16 apart
  constexpr int SP = 16, HALF = SP / SEG;            // HALF waves cover 4 SP band rows
  const uint32_t rows = (uint32_t)(nf + TILE_PAD);
  const __amdgpu_buffer_rsrc_t hrs = buf_rsrc(mv.tb, rows * PB);
  const __amdgpu_buffer_rsrc_t ors = buf_rsrc(mv.tb_off[CFG], rows * OB);
  const uint32_t lrow = (uint32_t)(w / HALF * 4 * SP + q * SP + w % HALF * SEG);
  const uint32_t hoff = lrow * PB + (uint32_t)l16 * 4u, ooff = lrow * OB + (uint32_t)(l16 % TILE_Q) * 4u;
  constexpr int NA = TILE_Q * 3 / 4;                 // registers of a record set: 4 of its 24 columns each
  float A[SEG][NA], U[2][TILE_Q][3];
  uint32_t O[SEG], at[TILE_Q];                       // O: lane r of a row holds the row's r-th block's offset
  auto fetch_off = [&](int t, int p) { O[t] = __builtin_amdgcn_raw_buffer_load_b32(ors, ooff, (uint32_t)(p + t) * OB, 0); };
  auto fetch_rec = [&](int t, int p) {
#pragma unroll
    for (int r = 0; r < NA; ++r)
      A[t][r] = __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(hrs, hoff + 64u * r, (uint32_t)(p + t) * PB, 0));
  };
  auto addresses = [&](int t) {                      // row_newbcast:r
    auto one = [&](auto rc) {
      constexpr int r = decltype(rc)::value;
      at[r] = lbase + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)O[t], 0x150 + r, 0xf, 0xf, true);
    };
    one(std::integral_constant<int, 0>()); one(std::integral_constant<int, 1>());
    one(std::integral_constant<int, 2>()); one(std::integral_constant<int, 3>());
    one(std::integral_constant<int, 4>()); one(std::integral_constant<int, 5>());
    one(std::integral_constant<int, 6>()); one(std::integral_constant<int, 7>());
  };
  auto read_u = [&](int ub, int g) {
#pragma unroll
    for (int r = 0; r < TILE_Q; ++r) {
      const lds_float* src = (const lds_float*)(uintptr_t)at[r];
#pragma unroll
      for (int c = 0; c < 3; ++c) U[ub][r][c] = src[5 * tile_stride(TILE_RING) * g + 3 * c];
    }
  };
  f4 Y[NG], Ysum[NG];                                // a chunk's products; the chunks before it
  float bacc[NG], bsum[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    Ysum[g] = f4{0.f, 0.f, 0.f, 0.f};
    bsum[g] = 0.f;
  }
  auto products = [&](int ub, const float (&a)[NA], int g) {
    const float(&u)[TILE_Q][3] = U[ub];
    // one 4-row column of H'' per instruction, column k in block k % 4 of
    // register k / 4; two chains, since a product waits for the last one of its
    f4 W = {0.f, 0.f, 0.f, 0.f}, X = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 3 * TILE_Q; k += 4) {
      W = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k / 4], u[k / 3][k % 3], W, 2, 0, 0);
      X = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k / 4], u[(k + 1) / 3][(k + 1) % 3], X, 2, 1, 0);
      W = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k / 4], u[(k + 2) / 3][(k + 2) % 3], W, 2, 2, 0);
      X = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k / 4], u[(k + 3) / 3][(k + 3) % 3], X, 2, 3, 0);
    }
    W += X;
#pragma unroll
    for (int r = 0; r < 3; ++r) Y[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[0][r], W[r], Y[g], 0, 0, 0);
    bacc[g] += W[3];
  };
#pragma unroll
  for (int t = 0; t < SEG; ++t) {
    fetch_off(t, pa);
    fetch_rec(t, pa);
  }
  uint32_t slot4 = 0;                                // bytes of the chunk's first ring slot
  __syncthreads();
  for (int p0 = pa; p0 < pb; p0 += CH) {
    // chunk p0 + CH needs positions up to p0 + R + CH: read them ahead; they
    // replace positions [p0, p0 + CH), which no later row reads
    const bool refill = p0 + R < nf && p0 + CH < pb;
    uint32_t pre[NP];
    addresses(0);
    read_u(0, 0);
    fetch_off(0, p0 + CH);
    if (refill) {
      const uint32_t f4b = tile_piece(p0 + R, 0) * 4u;
#pragma unroll
      for (int e = 0; e < NP; ++e) pre[e] = load_piece(gat[e] + f4b);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      Y[g] = f4{0.f, 0.f, 0.f, 0.f};
      bacc[g] = 0.f;
    }
    // phases (band row t, vertex group g): the U columns one phase ahead, the
    // next chunk's records and offsets once this one's are used up.  Loads
    // return in order, so nothing waits for the basis pieces (from HBM)
    // before the chunk's end.  The barriers keep the compiler from moving
    // the reads next to their uses.
#pragma unroll
    for (int f = 0; f < PHASES; ++f) {
      const int t = f / NG, g = f % NG;
      if (f + 1 < PHASES) {
        if (g + 1 == NG) addresses(t + 1);
        read_u((f + 1) & 1, (f + 1) % NG);
        if (g + 1 == NG) fetch_off(t + 1, p0 + CH);
      }
      __builtin_amdgcn_sched_barrier(0);
      products(f & 1, A[t], g);
      if (g + 1 == NG) fetch_rec(t, p0 + CH);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      Ysum[g] += Y[g];
      bsum[g] += bacc[g];
    }
    if (refill) {
      __syncthreads();                               // chunk p0's ring reads are done
#pragma unroll
      for (int e = 0; e < NP; ++e) put_piece(lat[e] + slot4, pre[e]);
      slot4 += (uint32_t)(CH * 36);
      if (slot4 == (uint32_t)(R * 36)) slot4 = 0;
      __syncthreads();
    }
  }
  __syncthreads();
  // Ht_i = Y + Y^T and b_i: sums over the waves (and for b the lane rows) in a
  // fixed order; lane l's Y[i] is entry (4 (l / 16) + i, l % 16) of a group's
  // 15 x 15 column products, of which the vertices' own 3 x 3 blocks are used
  float* red = smem;                                 // [NS][NG][5][64], the ring is free now
#pragma unroll
  for (int g = 0; g < NG; ++g) {
#pragma unroll
    for (int k = 0; k < 4; ++k) red[((w * NG + g) * 5 + k) * 64 + l] = Ysum[g][k];
    red[((w * NG + g) * 5 + 4) * 64 + l] = bsum[g];
  }
  __syncthreads();
  for (int e = tid; e < nv * NR; e += NT) {
    const int v = e / NR, k = e % NR, c3 = 3 * (v % 5);
    float acc = 0.f, acc_t = 0.f;
    for (int ww = 0; ww < NS; ++ww) {
      const float* rw = red + (ww * NG + v / 5) * 5 * 64;
      if (k < 9) {
        const int r = c3 + k / 3, c = c3 + k % 3;
        acc += rw[(r % 4) * 64 + (r / 4) * 16 + c];
        acc_t += rw[(c % 4) * 64 + (c / 4) * 16 + r];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) acc += rw[4 * 64 + r * 16 + c3 + k - 9];
      }
    }
    if (seg > 0) gptr_w(seg_sums<float, 3>(mv, seg, i0 + v))[k] = k < 9 ? acc + acc_t : acc;
    else if (k < 9) gptr_w(KL)[(size_t)(i0 + v) * 18 + 9 + k] = acc + acc_t;
    else if (bout != nullptr) gptr_w(bout)[(size_t)(k - 9) * mv.n + i0 + v] = double(acc);
  }
}

// With dout given, dout holds b_i on entry and receives dx_i = -K (g_i - L b_i)
// (the arithmetic of update_body).
template <typename T, int D>
__device__ __forceinline__ void dm_finish_body(const MeshView& mv, int method, int i,
                                               const T* __restrict__ hb, T* __restrict__ KL,
                                               unsigned long long* __restrict__ fb,
                                               const double* __restrict__ g, double* __restrict__ dout,
                                               const double* x, double* xtrial, int nseg) {
  constexpr int DD = D * D;
  T A[DD], Ht[DD], bs[D];
  const T* in = KL + (size_t)i * 2 * DD;
#pragma unroll
  for (int r = 0; r < DD; ++r) {
    A[r] = in[r];
    Ht[r] = in[DD + r];
  }
#pragma unroll
  for (int c = 0; c < D; ++c) bs[c] = T(0);
  for (int sg = 1; sg < nseg; ++sg) {                // the other segments' sums, in order
    const T* ss = seg_sums<T, D>(mv, sg, i);
#pragma unroll
    for (int r = 0; r < DD; ++r) Ht[r] += ss[r];
#pragma unroll
    for (int c = 0; c < D; ++c) bs[c] += ss[DD + c];
  }
  cc_finish<T, D>(mv, method, i, mv.nf <= 1, A, Ht, hb, KL, fb);
  if (dout == nullptr) return;
  const int n = mv.n;
  const T* kl = KL + (size_t)i * 2 * DD;
  T b[D], gt[D];
#pragma unroll
  for (int c = 0; c < D; ++c) b[c] = T(dout[(size_t)c * n + i]) + bs[c];
#pragma unroll
  for (int r = 0; r < D; ++r) {
    T lb = T(0);
#pragma unroll
    for (int l = 0; l < D; ++l) lb += kl[DD + r * D + l] * b[l];
    gt[r] = T(g[(size_t)r * n + i] - double(lb));
  }
#pragma unroll
  for (int r = 0; r < D; ++r) {
    T acc = T(0);
#pragma unroll
    for (int l = 0; l < D; ++l) acc += kl[r * D + l] * gt[l];
    dout[(size_t)r * n + i] = -double(acc);
    // the trial point x + d of this vertex (Jacobi: the batched path's axpy;
    // coloured sweep: x and xtrial are the same running state, moved in place)
    if (xtrial != nullptr) xtrial[(size_t)r * n + i] = x[(size_t)r * n + i] - double(acc);
  }
}

template <typename T, int D>
__global__ void __launch_bounds__(WG) k_cc_dm_finish(MeshView mv, int method, int v0, int v1,
                                                     const T* __restrict__ hb, T* __restrict__ KL,
                                                     unsigned long long* __restrict__ fb,
                                                     const double* __restrict__ g, double* __restrict__ dout,
                                                     const double* xfrom, double* xmove, int nseg) {
  const int i = v0 + blockIdx.x * WG + threadIdx.x;
  if (i < v1) dm_finish_body<T, D>(mv, method, i, hb, KL, fb, g, dout, xfrom, xmove, nseg);
}

template <typename T, int D, int TV, int CH>
__global__ void __launch_bounds__(CH) k_cc_prep_band(MeshView mv, int v0, int v1,
                                                      const T* __restrict__ hb, T* __restrict__ KL,
                                                      const double* __restrict__ g, double* __restrict__ bout,
                                                      int nseg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int nb = gridDim.x / nseg, i0 = v0 + blockIdx.x % nb * TV;
  prep_band_body<T, D, TV, CH>(mv, i0, min(TV, v1 - i0), hb, KL, reinterpret_cast<T*>(smem_raw), g,
                               bout, blockIdx.x / nb, nseg);
}

template <int NG, int NS, int CH>
__global__ void __launch_bounds__(64 * NS, 4)
k_cc_prep_tile(MeshView mv, int v0, int v1, const float* __restrict__ hb, float* __restrict__ KL,
               double* __restrict__ bout, int nseg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int nb = gridDim.x / nseg, i0 = v0 + blockIdx.x % nb * 5 * NG;
  prep_tile_body<NG, NS, CH>(mv, i0, min(5 * NG, v1 - i0), hb, KL, reinterpret_cast<float*>(smem_raw), bout,
                             blockIdx.x / nb, nseg);
}

// dx_i = -K_i (g_i - L_i U_i^T g_C); written to d (Jacobi) or added to x
// (coloured sweep).  G lanes per vertex share its support.
template <typename T, int D, int G>
__device__ __forceinline__ void update_body(const MeshView& mv, int method, int i, bool active,
                                            int lane, const T* __restrict__ KL,
                                            const double* __restrict__ g, double* out,
                                            int accumulate, const double* from = nullptr) {
  constexpr int DD = D * D;
  const T* Ub = basis_of<T>(mv);
  const int n = mv.n;
  T b[D];
#pragma unroll
  for (int c = 0; c < D; ++c) b[c] = T(0);
  if (active && method != 0) {
    int64_t sp0, sp1;
    supp_range(mv, i, sp0, sp1);
    for (int64_t q = sp0 + lane; q < sp1; q += G) {
      const int j = supp_vertex(mv, q, sp0);
      T gj[D];
#pragma unroll
      for (int c = 0; c < D; ++c) gj[c] = T(g[c * n + j]);
      if (mv.rot) {                               // (R_j U)^T g_j = U^T (R_j^T g_j)
        T t[D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
          T acc = T(0);
#pragma unroll
          for (int l = 0; l < D; ++l) acc += T(mv.rot[(size_t)j * DD + l * D + c]) * gj[l];
          t[c] = acc;
        }
#pragma unroll
        for (int c = 0; c < D; ++c) gj[c] = t[c];
      }
#pragma unroll
      for (int r = 0; r < D; ++r) {
        T acc = T(0);
#pragma unroll
        for (int l = 0; l < D; ++l) acc += Ub[q * DD + l * D + r] * gj[l];
        b[r] += acc;
      }
    }
  }
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1)
#pragma unroll
    for (int c = 0; c < D; ++c) b[c] += __shfl_xor(b[c], off, G);
  if (!active || lane != 0) return;
  const T* kl = KL + (size_t)i * 2 * DD;
  T gt[D];
#pragma unroll
  for (int r = 0; r < D; ++r) {
    T lb = T(0);
#pragma unroll
    for (int l = 0; l < D; ++l) lb += kl[DD + r * D + l] * b[l];
    gt[r] = T(g[r * n + i] - double(lb));
  }
#pragma unroll
  for (int r = 0; r < D; ++r) {
    T acc = T(0);
#pragma unroll
    for (int l = 0; l < D; ++l) acc += kl[r * D + l] * gt[l];
    if (from != nullptr) out[r * n + i] = from[r * n + i] - double(acc);
    else if (accumulate) out[r * n + i] -= double(acc);
    else out[r * n + i] = -double(acc);
  }
}

template <typename T, int D, int G>
__global__ void __launch_bounds__(WG) k_cc_update(MeshView mv, int method, int v0, int v1,
                                                  const T* __restrict__ KL,
                                                  const double* __restrict__ g,
                                                  double* out, int accumulate, const double* from) {
  const int i = v0 + blockIdx.x * (WG / G) + threadIdx.x / G;
  update_body<T, D, G>(mv, method, i, i < v1, threadIdx.x % G, KL, g, out, accumulate, from);
}

// Step energy: blocks [0, nbe) sum element energies, the rest the free-vertex
// inertia and gravity terms; one partial per block.
// Block b < nbe sums element energies, the others free-vertex terms.
template <int D, bool FCR>
__device__ __forceinline__ double energy_body(const MeshView& mv, int b, int nbe,
                                              const double* __restrict__ x,
                                              const double* __restrict__ xt, const Material& mat) {
  double v = 0.0;
  const int n = mv.n;
  if (b < nbe) {
    const int e = b * WG + threadIdx.x;
    if (e < mv.m) {
      double F[D][D], beta[D + 1][D], vol;
      load_element<double, D>(mv, e, x, F, beta, vol);
      v = mat.s_el * vol * material_psi<double, D>(F, mat.mu, mat.lam, FCR ? mat.model : MAT_SNH);
    }
  } else {
    const int j = (b - nbe) * WG + threadIdx.x;
    if (j < mv.nf) {
      const double mj = mv.mass[j];
      double in = 0.0, gr = 0.0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const double dx = x[c * n + j] - xt[c * n + j];
        in += dx * dx;
        gr += mat.grav[c] * x[c * n + j];
      }
      v = mat.w_in * 0.5 * mj * in - mat.s_el * mj * gr;
    }
  }
  return v;
}

// energy_body at the positions x + alpha d (formed as the trial-point update
// forms them), block for block.
template <int D, bool FCR>
__device__ __forceinline__ double energy_body_along(const MeshView& mv, int b, int nbe,
                                                    const double* __restrict__ x,
                                                    const double* __restrict__ d, double alpha,
                                                    const double* __restrict__ xt,
                                                    const Material& mat) {
  double v = 0.0;
  const int n = mv.n;
  if (b < nbe) {
    const int e = b * WG + threadIdx.x;
    if (e < mv.m) {
      double F[D][D], beta[D + 1][D], vol;
      load_element_along<double, D>(mv, e, x, d, alpha, F, beta, vol);
      v = mat.s_el * vol * material_psi<double, D>(F, mat.mu, mat.lam, FCR ? mat.model : MAT_SNH);
    }
  } else {
    const int j = (b - nbe) * WG + threadIdx.x;
    if (j < mv.nf) {
      const double mj = mv.mass[j];
      double in = 0.0, gr = 0.0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const double p = x[c * n + j] + alpha * d[c * n + j];
        const double dx = p - xt[c * n + j];
        in += dx * dx;
        gr += mat.grav[c] * p;
      }
      v = mat.w_in * 0.5 * mj * in - mat.s_el * mj * gr;
    }
  }
  return v;
}

template <int D, bool FCR>
__global__ void __launch_bounds__(WG) k_energy(MeshView mv, const double* __restrict__ x,
                                               const double* __restrict__ xt, Material mat,
                                               int nbe, double* __restrict__ partials) {
  __shared__ double red[WG];
  const double v = energy_body<D, FCR>(mv, blockIdx.x, nbe, x, xt, mat);
  const double tot = block_sum<WG>(v, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// Step energy (blocks [0, ne)) and gradient (the rest) at x in one launch: an
// accepted trial point needs both, and each alone is a few us of mostly
// latency on a small mesh.  With one reduction into host memory per point and
// no second gradient at the point that the next sweep starts from, an iteration
// of a single mesh is 6 launches and 1 wait instead of 13 and 2: the step of a
// 17x17 square took 963 us and takes 594, of a 41x2x2 rod 466 and 252, of a
// 21x6x6 bar 508 and 328, of the 81x21x21 beam with patch bases 2343 and 1768.
template <int D, int G, bool FCR>
__global__ void __launch_bounds__(WG) k_energy_grad(MeshView mv, const double* __restrict__ x,
                                                    const double* __restrict__ xt, Material mat, int nbe, int ne,
                                                    double* __restrict__ g, double* __restrict__ partials) {
  __shared__ double red[WG];
  const int b = blockIdx.x;
  double v;
  if (b < ne)
    v = energy_body<D, FCR>(mv, b, nbe, x, xt, mat);
  else
    v = gradient_body<D, G, FCR>(mv, grad_vertex(mv, (b - ne) * (WG / G) + threadIdx.x / G), threadIdx.x % G, x, xt,
                                 mat, g);
  const double tot = block_sum<WG>(v, red);
  if (threadIdx.x == 0) partials[b] = tot;
}

// out[0] = sum of partials[0, ne), out[1] = sum of partials[ne, ne + ng), one
// block each (the first block stands for sum `first`, so one block can do
// either alone), and the step's counters into out[2 ..].  out may be pinned
// host memory: the caller then reads it after one synchronisation, without a
// copy of its own (about 3 us on the stream) for each value.
__global__ void __launch_bounds__(WG) k_reduce_eg(const double* __restrict__ partials, int ne, int ng, int first,
                                                  const unsigned long long* __restrict__ counters, int nc,
                                                  double* __restrict__ out) {
  __shared__ double red[WG];
  const int which = first + blockIdx.x;
  const double* p = partials + (which ? ne : 0);
  const int cnt = which ? ng : ne;
  double v = 0.0;
  for (int i = threadIdx.x; i < cnt; i += WG) v += p[i];
  const double tot = block_sum<WG>(v, red);
  if (threadIdx.x == 0) out[which] = tot;
  if (blockIdx.x == 0 && (int)threadIdx.x < nc)
    reinterpret_cast<unsigned long long*>(out)[2 + threadIdx.x] = counters[threadIdx.x];
}

__global__ void k_axpy(int count, const double* __restrict__ x, const double* __restrict__ d,
                       double alpha, double* __restrict__ out) {
  const int t = blockIdx.x * WG + threadIdx.x;
  if (t < count) out[t] = x[t] + alpha * d[t];
}

template <int D>
__global__ void k_predict(MeshView mv, const int* __restrict__ vperm,
                          const double* __restrict__ xu, const double* __restrict__ vu,
                          const double* __restrict__ xbc, double h, int quasi,
                          double* __restrict__ x, double* __restrict__ xt,
                          double* __restrict__ x0, double* __restrict__ xtrial, int* __restrict__ bad) {
  const int v = blockIdx.x * WG + threadIdx.x;
  if (v >= mv.n) return;
  const int u = vperm[v], n = mv.n;
  bool ok = true;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const double xp = xu[u * D + c], vp = vu[u * D + c];
    ok = ok && isfinite(xp) && isfinite(vp);
    x0[c * n + v] = xp;
    double xh;
    if (v < mv.nf) {
      xh = quasi ? xp : xp + h * vp;
    } else {
      xh = xbc ? xbc[u * D + c] : xp;
      ok = ok && isfinite(xh);
    }
    xt[c * n + v] = xh;
    x[c * n + v] = xh;
    // the trial buffer too: a sweep writes its free entries only
    xtrial[c * n + v] = xh;
  }
  if (!ok) atomicOr(bad, 1);
}

template <int D>
__global__ void k_finalize(MeshView mv, const int* __restrict__ vperm, const double* __restrict__ x,
                           const double* __restrict__ xt, const double* __restrict__ x0, double h, int quasi,
                           double* __restrict__ xu, double* __restrict__ vu) {
  const int v = blockIdx.x * WG + threadIdx.x;
  if (v >= mv.n) return;
  const int u = vperm[v], n = mv.n;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const double xn = x[c * n + v];
    xu[u * D + c] = xn;
    vu[u * D + c] = quasi ? 0.0 : (xn - x0[c * n + v]) / h;
    if (mv.corr) mv.corr[c * n + v] = v < mv.nf ? xn - xt[c * n + v] : 0.0;
  }
}

template <int D>
__global__ void k_gather_user(MeshView mv, const int* __restrict__ vinv, const double* __restrict__ src,
                              double* __restrict__ dst) {
  const int u = blockIdx.x * WG + threadIdx.x;
  if (u >= mv.n) return;
  const int v = vinv[u];
#pragma unroll
  for (int c = 0; c < D; ++c) dst[c * mv.n + v] = src[u * D + c];
}

template <int D>
__global__ void k_scatter_user(MeshView mv, const int* __restrict__ vperm, const double* __restrict__ src,
                               double* __restrict__ dst, int free_only) {
  const int v = blockIdx.x * WG + threadIdx.x;
  if (v >= mv.n) return;
  const int u = vperm[v];
  const bool keep = !free_only || v < mv.nf;
#pragma unroll
  for (int c = 0; c < D; ++c) dst[u * D + c] = keep ? src[c * mv.n + v] : 0.0;
}

// Parity probe: element gradients (float64 or T) and the full (un-packed)
// Hessian blocks in caller element order.
template <typename T, int D>
__global__ void k_probe_elem(MeshView mv, const double* __restrict__ x, const int* __restrict__ eperm,
                             const T* __restrict__ est, T mu, T lam, int model, double* __restrict__ ge,
                             double* __restrict__ He) {
  constexpr int K = D + 1, DD = D * D;
  const int e = blockIdx.x * WG + threadIdx.x;
  if (e >= mv.m) return;
  const int eu = eperm[e];
  T F[D][D], beta[K][D], vol, P[D][D];
  load_element<T, D>(mv, e, x, F, beta, vol);
  material_pk1<T, D>(F, mu, lam, model, P);
  for (int a = 0; a < K; ++a)
    for (int r = 0; r < D; ++r) {
      T s = T(0);
      for (int q = 0; q < D; ++q) s += P[r][q] * beta[a][q];
      ge[((size_t)eu * K + a) * D + r] = double(vol * s);
    }
  const int m = mv.m;
  for (int a = 0; a < K; ++a)
    for (int b = 0; b < K; ++b) {
      const int p = a <= b ? pidx<K>(a, b) : pidx<K>(b, a);
      const T* blk = est + ((size_t)p * m + e) * DD;
      for (int r = 0; r < D; ++r)
        for (int s = 0; s < D; ++s)
          He[(((size_t)eu * K + a) * K + b) * DD + r * D + s] =
              double(a <= b ? blk[r * D + s] : blk[s * D + r]);
    }
}

// ---------------------------------------------------------------------------
static inline int nblocks(long long n, int per) { return (int)((n + per - 1) / per); }

#define CC_DISPATCH_D(D_, ...)                     \
  do {                                             \
    if ((D_) == 2) { constexpr int D = 2; __VA_ARGS__; } \
    else { constexpr int D = 3; __VA_ARGS__; }     \
  } while (0)

// Material-dependent kernels come in two builds: FCR = false compiles the
// stable neo-Hookean path alone (its register budget untouched by the
// Fixed Corotational SVD); FCR = true follows each mesh's model at run time.
#define CC_DISPATCH_MAT(any_fcr, ...)                          \
  do {                                                         \
    if (any_fcr) { constexpr bool FCR = true; __VA_ARGS__; }   \
    else { constexpr bool FCR = false; __VA_ARGS__; }          \
  } while (0)

void launch_predict(const MeshView& mv, const int* vperm, const double* x_user, const double* v_user,
                    const double* x_bc, double h, int quasi, double* x, double* xt, double* x0,
                    double* xtrial, int* bad, hipStream_t s) {
  CC_DISPATCH_D(mv.D, k_predict<D><<<nblocks(mv.n, WG), WG, 0, s>>>(mv, vperm, x_user, v_user, x_bc,
                                                                   h, quasi, x, xt, x0, xtrial, bad));
}

void launch_finalize(const MeshView& mv, const int* vperm, const double* x, const double* xt, const double* x0,
                     double h, int quasi, double* x_user, double* v_user, hipStream_t s) {
  CC_DISPATCH_D(mv.D, k_finalize<D><<<nblocks(mv.n, WG), WG, 0, s>>>(mv, vperm, x, xt, x0, h, quasi,
                                                                    x_user, v_user));
}

void launch_elem_hess_list(const MeshView& mv, int prec, const double* x, const Material& mat,
                           double scale, void* estore, hipStream_t s, const int* elist, int count) {
  if (count <= 0) return;
  const int nb = nblocks(count, EWG);
  if (prec == 0)
    CC_DISPATCH_MAT(mat.model == MAT_FCR,
                    CC_DISPATCH_D(mv.D, k_elem_hess<double, D, FCR><<<nb, elem_threads<double>(), 0, s>>>(
                                            mv, x, mat.mu, mat.lam, mat.model, scale, (double*)estore, elist,
                                            count)));
  else
    CC_DISPATCH_MAT(mat.model == MAT_FCR,
                    CC_DISPATCH_D(mv.D, k_elem_hess<float, D, FCR><<<nb, elem_threads<float>(), 0, s>>>(
                                            mv, x, (float)mat.mu, (float)mat.lam, mat.model, (float)scale,
                                            (float*)estore, elist, count)));
}

void launch_elem_hess(const MeshView& mv, int prec, const double* x, const Material& mat,
                      double scale, void* estore, hipStream_t s) {
  launch_elem_hess_list(mv, prec, x, mat, scale, estore, s, nullptr, mv.m);
}

void launch_assemble(const MeshView& mv, int prec, const void* estore, const Material& mat,
                     void* hb, const double* g, hipStream_t s) {
  launch_assemble_list(mv, prec, estore, mat, hb, g, s, nullptr, mv.nnzb);
}

void launch_assemble_list(const MeshView& mv, int prec, const void* estore, const Material& mat, void* hb,
                          const double* g, hipStream_t s, const int* slist, int count) {
  if (count <= 0) return;
  const int nb = nblocks(count, EWG);
  if (prec == 0)
    CC_DISPATCH_D(mv.D, k_assemble<double, D><<<nb, EWG, 0, s>>>(mv, (const double*)estore, mat.w_in,
                                                               (double*)hb, g, slist, count));
  else
    CC_DISPATCH_D(mv.D, k_assemble<float, D><<<nb, EWG, 0, s>>>(mv, (const float*)estore, (float)mat.w_in,
                                                              (float*)hb, g, slist, count));
}

constexpr int GRAD_G = 16;   // lanes per vertex of the gradient: a 3D star holds about 24 elements

int reduce_partials_capacity(const MeshView& mv) {
  // energy partials followed by gradient partials (kb_energy_grad)
  const int a = nblocks(mv.nf, WG / GRAD_G);
  const int b = nblocks(mv.m, WG) + nblocks(mv.nf, WG);
  return a + b + 1;
}

void launch_gradient(const MeshView& mv, const double* x, const double* xt, const Material& mat,
                     double* g, double* partials, int* nparts, hipStream_t s) {
  const int nb = nblocks(mv.nf, WG / GRAD_G);
  *nparts = nb;
  if (nb == 0) return;
  CC_DISPATCH_MAT(mat.model == MAT_FCR,
                  CC_DISPATCH_D(mv.D, k_gradient<D, GRAD_G, FCR><<<nb, WG, 0, s>>>(mv, x, xt, mat, g, partials)));
}

// LDS of the staged support rows per workgroup: 32 KB keeps five 256-thread
// workgroups per CU.  Longer rows are read from global memory instead.
constexpr size_t SPARSE_STAGE_MAX = 32 * 1024;

static int sparse_stage_cap(int supp, int G, int D, int prec) {
  const size_t bytes = (size_t)(WG / G) * supp * D * D * (prec == 0 ? 8 : 4);
  return supp > 0 && bytes <= SPARSE_STAGE_MAX ? supp : 0;
}

static size_t sparse_stage_bytes(int cap, int G, int D, int prec) {
  return (size_t)(WG / G) * cap * D * D * (prec == 0 ? 8 : 4);
}

template <typename T, int D>
static void prep_g(const MeshView& mv, int method, int v0, int v1, const void* hb, void* KL,
                   unsigned long long* fb, int G, hipStream_t s) {
  const int cnt = v1 - v0;
  const int prec = sizeof(T) == 8 ? 0 : 1;
  const int cap = sparse_stage_cap(mv.smap ? mv.smap_supp : 0, G, D, prec);
  const size_t lds = sparse_stage_bytes(cap, G, D, prec);
  if (G == 64)
    k_cc_prep<T, D, 64><<<nblocks(cnt, WG / 64), WG, lds, s>>>(mv, method, v0, v1, (const T*)hb,
                                                               (T*)KL, fb, cap);
  else
    k_cc_prep<T, D, 16><<<nblocks(cnt, WG / 16), WG, lds, s>>>(mv, method, v0, v1, (const T*)hb,
                                                               (T*)KL, fb, cap);
}

static int support_lanes(const MeshView& mv) {
  if (mv.dense_supp) return 64;
  const double avg = mv.nf > 0 ? double(mv.nnzb) / mv.nf : 0.0;  // proxy: row length
  (void)avg;
  return 16;
}

static size_t g_lds_limit = 64 * 1024;

void set_lds_limit(size_t bytes) { g_lds_limit = bytes; }

int band_ring(int nf, int band_w, int ch) {
  if (nf <= 0) return 0;
  return std::min(nf, ch + band_w);
}

// Resident waves per SIMD that the registers of the dense condensation allow
// (gfx950 builds of prep_band_body, 3D: float32 228 / 182 / 122 / 79 VGPRs
// for 4 / 3 / 2 / 1 rows, float64 226 / 149 for 2 / 1 rows)
static int dense_reg_waves(int prec, int tv) {
  if (prec == 0) return tv >= 2 ? 2 : 3;
  return tv >= 3 ? 2 : tv == 2 ? 4 : 6;
}

size_t dense_lds_bytes(int tv, int ring, int D, int prec, int ch) {
  const size_t S = prec == 0 ? 8 : 4;
  // ring slots (ring_slot_words), then the per-wave partial sums
  return (size_t)ring * ring_slot_words(tv, D, (int)S) * 4 + (size_t)(ch / 64) * tv * (D * D + D) * S;
}

// float64 keeps at most two rows per workgroup (the register file of 2
// waves/SIMD holds the accumulators of two float64 rows, four float32 ones).
// Among chunks that leave as many waves resident, the smallest wins: more,
// shorter workgroups fill the last round of a launch better.  With the rows
// chosen automatically, the most rows that still let two workgroups share a
// CU come first (one workgroup's barriers and ring fill then overlap the
// other's products); only when no row count allows two does one per CU do.
DenseCfg dense_config(const int* nf, const int* band_w, int count, int D, int prec, int cap, int chunk) {
  DenseCfg best;
  const int top = std::min(prec == 0 ? 2 : 4, cap > 0 ? cap : 4);
  for (int pass = cap > 0 ? 1 : 0; pass < 2 && best.tv == 0; ++pass)
    for (int tv = top; tv >= 1 && best.tv == 0; --tv) {
      int best_waves = 0;
      for (int ch : {128, 256, BWG}) {
        if (chunk > 0 && ch != chunk) continue;
        int ring = 0;
        for (int m = 0; m < count; ++m) ring = std::max(ring, band_ring(nf[m], band_w[m], ch));
        if (ring <= 0) continue;
        const size_t lds = dense_lds_bytes(tv, ring, D, prec, ch);
        if (lds > g_lds_limit || (pass == 0 && 2 * lds > g_lds_limit)) continue;
        const int waves = std::min((int)(g_lds_limit / lds) * (ch / 64), 4 * dense_reg_waves(prec, tv));
        if (waves > best_waves) {
          best_waves = waves;
          best.tv = tv;
          best.ch = ch;
          best.lds = lds;
        }
      }
    }
  return best;
}

// Workgroups of the dense condensation that are resident at once.
static int dense_resident(const DenseCfg& dc, int prec) {
  const int by_lds = (int)(g_lds_limit / dc.lds), by_reg = 4 * dense_reg_waves(prec, dc.tv) / (dc.ch / 64);
  return 256 * std::max(1, std::min(by_lds, by_reg));
}
static int tile_resident(int cfg) { return cfg == 2 ? 256 : 512; }

// Segments that a launch of the dense condensation splits its rows' bands
// into (rows: the band rows of all its workgroups): two up to one and a half times
// what the resident places do in the longest row's time, where a row is longer
// than a segment's unit (ring or chunk).  The time of such a launch is that of one
// workgroup's serial walk along the band, or two where the second round is mostly
// empty; half the walk costs a second ring fill.  In float32 the band kernel, whose
// places share a CU's issue, gains nothing where one round is more than half full.
// Unsplit / split, condensation and finish, us: band kernel, four vertices a
// workgroup on 1,024 places, 29x9x7 bars, one (441) 76 / 54, two (882) 90 / 94, three
// (1,323) 160 / 146; 21x6x6, one (180) 37 / 28, four (720) 48 / 52, six (1,080) 74 / 65;
// coloured step of ten uneven bars (0.43 of a round by rows, 0.78 by workgroups)
// 2248 / 2035; float64 21x6x6 bar's step 477 / 433 (three segments 452), coloured
// 17x17x17 cube (0.56 of a round) 2608 / 2514.  Tiles, steps of uneven bars, four
// (0.98 of a round by rows) 1386 / 1219, six (1.13) 1443 / 1343.
static int prep_segments(bool band32, int max_nf, long long rows, int unit, int resident) {
  const long long full = (long long)resident * max_nf;   // every place busy for the longest row's time
  const bool one_round = 2 * rows > full && rows <= full;
  return 2 * rows <= 3 * full && !(band32 && one_round) && max_nf > unit ? SEG_MAX : 1;
}

size_t tile_lds_bytes(int cfg, int nf, int band_w) {
  const int v = 5 * TILE_G[cfg - 1];
  const size_t ring = (size_t)v * tile_stride(tile_ring(cfg, nf, band_w)) * 4;
  return std::max(ring, (size_t)TILE_WAVES[cfg - 1] * v * 64 * 4);   // the final sums reuse the ring
}

// Ten vertices per workgroup share each record load and give two workgroups
// of eight waves per CU; below 400 such workgroups (a launch that does not
// fill the chip twice: a single bar, or one colour of a coloured sweep) five
// vertices spread further: the 29x9x7 bar's 353 five-vertex workgroups take 67
// us, in sixteen waves each (one per CU) 86 us.  Where the band leaves one
// workgroup per CU (the beam: 138 KB), it has sixteen waves.
int tile_config(const int* nf, const int* band_w, const int* rows, int count) {
  size_t lds[TILE_N + 1] = {};
  long long wgs = 0;
  bool ring = true;
  for (int m = 0; m < count; ++m) {
    for (int c = 1; c <= TILE_N; ++c) lds[c] = std::max(lds[c], tile_lds_bytes(c, nf[m], band_w[m]));
    ring = ring && (band_w[m] + TILE_CH[0] <= TILE_RING || nf[m] <= TILE_RING);
    wgs += nblocks(rows[m], 10);
  }
  if (ring && 2 * lds[1] <= g_lds_limit && wgs >= 400) return 1;
  if (2 * lds[3] <= g_lds_limit) return 3;
  return lds[2] <= g_lds_limit ? 2 : lds[3] <= g_lds_limit ? 3 : 0;
}

// Whether a launch of `blocks` workgroups (with that many band rows and ring
// positions between them) is long enough for the tiles: below that, the band
// kernel's smaller rings fill sooner, and its rows split better.
// Tiles / band kernel, condensation and finish, us: 21x6x6 bars, one 38 / 28, four
// 72 / 48; 29x9x7, one 72 / 54, two 121 / 90, three (530 workgroups of ten vertices)
// 156 / 145, four (706) 196 / 198 and corotated 186 / 206; 41x11x11, one (484, rows of
// 25 rings) 304 / 335; corotated 25x15x15 (1,080 of five, 14 rings) 459 / 476, 41x13x13
// (1,352, 18 rings) 642 / 741.  Steps of uneven corotated batches, three bars (425 of
// ten) 1141 / 1110, four (582) 1226 / 1289, six (720) 1351 / 1414, sixteen 3196 / 3492,
// 64 13121 / 13613; coloured, sixteen bars (294) 4849 / 4789, thirty (600) 8029 / 8467.
static bool tile_fills(int cfg, int blocks, long long rows, long long rings) {
  if (cfg == 1) return 10 * blocks >= 11 * tile_resident(1) || rows >= 12 * rings;
  return blocks >= 3 * tile_resident(cfg) || (cfg == 3 && blocks >= 700 && rows >= 16 * rings);
}

// Whether the band kernel is the better one for a mesh's share of such a launch in
// configuration cfg, given that it has every wave its registers allow: where rows
// are short enough for the tile's first ring fill to show, or without corotation,
// since rotating the gradient costs the band kernel, whose records do not carry it.
// The fill is not overlapped where one workgroup is on a CU (configuration 2), and
// costs most where rounding up to whole chunks leaves a quarter of the ring unused
// (3).  Full launches of equal bars, tiles / band kernel, condensation and finish,
// us, corotated: section 17x17, nf 4,913 2347 / 2023, 6,647 2595 / 2532, 10,115 2955 /
// 3067; 18x18 (band kernel short of waves), 5,832 2514 / 3692; 21x21, 3,528 653 / 580,
// 10,584 3248 / 3659; 13x13, 2,028 797 / 810, 6,760 2411 / 2655; step of seventeen
// 13x12x12 (ring of 384, 272 needed) 3496 / 3401.  Without: 17x17, 10,115 2961 / 2722,
// 17,340 4514 / 4191; 12x12, 5,760 2318 / 2138; 13x13, 6,760 2591 / 2377.
static bool band_better(const MeshView& mv, int cfg, bool corotate) {
  const int R = tile_ring(cfg, mv.nf, mv.band_w);
  if (cfg == 1) return false;
  if (corotate && (mv.nf >= 10 * R || (cfg == 3 && 4 * (TILE_CH[2] + mv.band_w) > 3 * R))) return false;
  const DenseCfg dc = dense_config(&mv.nf, &mv.band_w, 1, 3, 1);
  return dc.tv > 0 && dense_resident(dc, 1) / 256 * (dc.ch / 64) == 4 * dense_reg_waves(1, dc.tv);
}

bool tile_usable(const MeshView& mv, int prec, int tv_cap, int chunk) {
  if (prec != 1 || mv.D != 3 || tv_cap != 0 || chunk != 0 || mv.tb == nullptr || !mv.dense_supp || mv.nf < 2)
    return false;
  return tile_config(&mv.nf, &mv.band_w, &mv.nf, 1) > 0;
}

bool tile_chosen(const MeshView& mv, int prec, int tv_cap, int chunk, bool corotate, int rows) {
  if (!tile_usable(mv, prec, tv_cap, chunk)) return false;
  const int cfg = tile_config(&mv.nf, &mv.band_w, &rows, 1);
  return tile_fills(cfg, nblocks(rows, 5 * TILE_G[cfg - 1]), mv.nf, tile_ring(cfg, mv.nf, mv.band_w)) &&
         !band_better(mv, cfg, corotate);
}

#define CC_DISPATCH_TILE(cfg, ...)                                                    \
  do {                                                                                \
    if ((cfg) == 1) { constexpr int NG = 2, NS = 8, CH = 64; __VA_ARGS__; }           \
    else if ((cfg) == 2) { constexpr int NG = 1, NS = 16, CH = 256; __VA_ARGS__; }    \
    else { constexpr int NG = 1, NS = 8, CH = 128; __VA_ARGS__; }                     \
  } while (0)

#define CC_DISPATCH_TVCH(tv, ch, ...)                                                 \
  switch ((tv) * 1000 + (ch)) {                                                       \
    case 1128: { constexpr int TV = 1, CH = 128; __VA_ARGS__; } break;                \
    case 2128: { constexpr int TV = 2, CH = 128; __VA_ARGS__; } break;                \
    case 3128: { constexpr int TV = 3, CH = 128; __VA_ARGS__; } break;                \
    case 4128: { constexpr int TV = 4, CH = 128; __VA_ARGS__; } break;                \
    case 1256: { constexpr int TV = 1, CH = 256; __VA_ARGS__; } break;                \
    case 2256: { constexpr int TV = 2, CH = 256; __VA_ARGS__; } break;                \
    case 3256: { constexpr int TV = 3, CH = 256; __VA_ARGS__; } break;                \
    case 4256: { constexpr int TV = 4, CH = 256; __VA_ARGS__; } break;                \
    case 1512: { constexpr int TV = 1, CH = 512; __VA_ARGS__; } break;                \
    case 2512: { constexpr int TV = 2, CH = 512; __VA_ARGS__; } break;                \
    case 3512: { constexpr int TV = 3, CH = 512; __VA_ARGS__; } break;                \
    default: { constexpr int TV = 4, CH = 512; __VA_ARGS__; } break;                  \
  }

// True when the mesh's dense basis can be streamed through the LDS ring in
// this precision (float64 needs the float64 copy of the basis).
static bool band_ok(const MeshView& mv, int prec) {
  if (!mv.dense_supp || mv.hq == nullptr || mv.nf < 2) return false;
  if (prec == 0 && mv.U_d == nullptr) return false;
  return dense_config(&mv.nf, &mv.band_w, 1, mv.D, prec).tv > 0;
}

template <typename T, int D>
static bool prep_dense(const MeshView& mv, int prec, int method, int v0, int v1, const void* hb,
                       void* KL, unsigned long long* fb, const double* g, double* dout, double* xmove,
                       const double* xfrom, int tv_cap, int chunk, hipStream_t s) {
  if (method == 0 || !band_ok(mv, prec)) return false;
  if constexpr (sizeof(T) == 4 && D == 3)
    if (mv.tile) {
      const int rows = v1 - v0, cfg = tile_config(&mv.nf, &mv.band_w, &rows, 1);
      const int blocks = nblocks(rows, 5 * TILE_G[cfg - 1]);
      const int nseg = prep_segments(false, mv.nf, (long long)blocks * mv.nf, tile_ring(cfg, mv.nf, mv.band_w),
                                     tile_resident(cfg));
      CC_DISPATCH_TILE(cfg, k_cc_prep_tile<NG, NS, CH><<<blocks * nseg, 64 * NS,
                                                       tile_lds_bytes(cfg, mv.nf, mv.band_w), s>>>(
                                mv, v0, v1, (const float*)hb, (float*)KL, g != nullptr ? dout : nullptr, nseg));
      k_cc_dm_finish<T, D><<<nblocks(v1 - v0, WG), WG, 0, s>>>(mv, method, v0, v1, (const T*)hb, (T*)KL, fb,
                                                              g, dout, xfrom != nullptr ? xfrom : xmove,
                                                              g != nullptr ? xmove : nullptr, nseg);
      return true;
    }
  // one colour's rows in float32: chunks of 256, as in a batch's coloured sweeps
  // (41x11x11 bar, two iterations, 128 / 256: 2014 / 1618 us; float64 2518 / 2718)
  DenseCfg dc{};
  if (prec == 1 && chunk == 0 && v1 - v0 < mv.nf) dc = dense_config(&mv.nf, &mv.band_w, 1, D, prec, tv_cap, 256);
  if (dc.tv == 0) dc = dense_config(&mv.nf, &mv.band_w, 1, D, prec, tv_cap, chunk);
  if (dc.tv == 0) return false;
  const int blocks = nblocks(v1 - v0, dc.tv);
  const int nseg = prep_segments(prec == 1, mv.nf, (long long)blocks * mv.nf, dc.ch, dense_resident(dc, prec));
  CC_DISPATCH_TVCH(dc.tv, dc.ch, k_cc_prep_band<T, D, TV, CH><<<blocks * nseg, CH, dc.lds, s>>>(
                                     mv, v0, v1, (const T*)hb, (T*)KL, g, dout, nseg));
  k_cc_dm_finish<T, D><<<nblocks(v1 - v0, WG), WG, 0, s>>>(mv, method, v0, v1, (const T*)hb, (T*)KL, fb,
                                                          g, dout, xfrom != nullptr ? xfrom : xmove,
                                                          g != nullptr ? xmove : nullptr, nseg);
  return true;
}

bool launch_cc_prep(const MeshView& mv, int prec, int method, int v0, int v1, const void* hb,
                    void* KL, unsigned long long* fb, hipStream_t s, const double* g, double* dout,
                    double* xmove, int tv_cap, int chunk, const double* xfrom) {
  if (v1 <= v0) return g != nullptr;
  bool done = false;
  if (prec == 0)
    CC_DISPATCH_D(mv.D, done = prep_dense<double, D>(mv, prec, method, v0, v1, hb, KL, fb, g, dout, xmove,
                                                     xfrom, tv_cap, chunk, s));
  else
    CC_DISPATCH_D(mv.D, done = prep_dense<float, D>(mv, prec, method, v0, v1, hb, KL, fb, g, dout, xmove,
                                                    xfrom, tv_cap, chunk, s));
  if (done) return g != nullptr;
  const int G = support_lanes(mv);
  if (prec == 0) CC_DISPATCH_D(mv.D, prep_g<double, D>(mv, method, v0, v1, hb, KL, fb, G, s));
  else CC_DISPATCH_D(mv.D, prep_g<float, D>(mv, method, v0, v1, hb, KL, fb, G, s));
  return false;
}

template <typename T, int D>
static void update_g(const MeshView& mv, int method, int v0, int v1, const void* KL, const double* g,
                     double* out, int acc, const double* from, int G, hipStream_t s) {
  const int cnt = v1 - v0;
  if (G == 64)
    k_cc_update<T, D, 64><<<nblocks(cnt, WG / 64), WG, 0, s>>>(mv, method, v0, v1, (const T*)KL, g,
                                                               out, acc, from);
  else
    k_cc_update<T, D, 16><<<nblocks(cnt, WG / 16), WG, 0, s>>>(mv, method, v0, v1, (const T*)KL, g,
                                                               out, acc, from);
}

void launch_cc_update(const MeshView& mv, int prec, int method, int v0, int v1, const void* KL,
                      const double* g, double* x_or_d, int accumulate, hipStream_t s,
                      const double* from) {
  if (v1 <= v0) return;
  const int G = support_lanes(mv);
  if (prec == 0)
    CC_DISPATCH_D(mv.D, update_g<double, D>(mv, method, v0, v1, KL, g, x_or_d, accumulate, from, G, s));
  else
    CC_DISPATCH_D(mv.D, update_g<float, D>(mv, method, v0, v1, KL, g, x_or_d, accumulate, from, G, s));
}

void launch_energy(const MeshView& mv, const double* x, const double* xt, const Material& mat,
                   double* partials, int* nparts, hipStream_t s) {
  const int nbe = nblocks(mv.m, WG), nbv = nblocks(mv.nf, WG);
  *nparts = nbe + nbv;
  if (nbe + nbv == 0) return;
  CC_DISPATCH_MAT(mat.model == MAT_FCR,
                  CC_DISPATCH_D(mv.D, k_energy<D, FCR><<<nbe + nbv, WG, 0, s>>>(mv, x, xt, mat, nbe, partials)));
}


// R_j = U V^T from the rotation-variant SVD of
// M = sum_{k in N(j)} (x_k - x_j)(X_k - X_j)^T: the polar rotation (det +1).
template <int D>
__device__ __forceinline__ void rotation_body(const MeshView& mv, int j, const double* __restrict__ x,
                                              const int* __restrict__ nptr, const int* __restrict__ nidx,
                                              const double* __restrict__ Xr, double* __restrict__ rot) {
  if (j >= mv.nf) return;
  const int n = mv.n;
  double M[D][D];
#pragma unroll
  for (int r = 0; r < D; ++r)
#pragma unroll
    for (int c = 0; c < D; ++c) M[r][c] = 0.0;
  double xj[D], Xj[D];
#pragma unroll
  for (int c = 0; c < D; ++c) { xj[c] = x[(size_t)c * n + j]; Xj[c] = Xr[(size_t)c * n + j]; }
  for (int t = nptr[j]; t < nptr[j + 1]; ++t) {
    const int k = nidx[t];
    double dx[D], dX[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      dx[c] = x[(size_t)c * n + k] - xj[c];
      dX[c] = Xr[(size_t)c * n + k] - Xj[c];
    }
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c) M[r][c] += dx[r] * dX[c];
  }
  double U[D][D], V[D][D], sig[D];
  svd_rv<double, D>(M, U, V, sig);
#pragma unroll
  for (int r = 0; r < D; ++r)
#pragma unroll
    for (int c = 0; c < D; ++c) {
      double acc = 0.0;
#pragma unroll
      for (int l = 0; l < D; ++l) acc += U[r][l] * V[c][l];
      rot[(size_t)j * D * D + r * D + c] = acc;
    }
}

template <int D>
__global__ void __launch_bounds__(WG) k_rotations(MeshView mv, const double* __restrict__ x,
                                                  const int* __restrict__ nptr, const int* __restrict__ nidx,
                                                  const double* __restrict__ Xr, double* __restrict__ rot) {
  rotation_body<D>(mv, blockIdx.x * WG + threadIdx.x, x, nptr, nidx, Xr, rot);
}

void launch_rotations(const MeshView& mv, const double* x, const int* nptr, const int* nidx,
                      const double* Xr, double* rot, hipStream_t s) {
  if (mv.nf <= 0 || !x || !nptr || !nidx || !Xr || !rot) return;
  CC_DISPATCH_D(mv.D, k_rotations<D><<<nblocks(mv.nf, WG), WG, 0, s>>>(mv, x, nptr, nidx, Xr, rot));
}

// What a sweep needs at a point before its assembly, in one launch: vertex
// rotations (rot given), element Hessians (of the list or all) and the gradient
// (g given).  None reads another's result, and on a mesh or batch that does not
// fill the chip each is one long chain of dependent loads and float64
// arithmetic per thread (11 to 15 us), so side by side they take little more
// than the longest.  Block b: rotations first, which take longest, with as few
// threads per workgroup as the elements, then elements, then gradient.
// Measured, one by one and in one launch: directions of the corotated 29x9x7 bar 188
// and 164 us; coloured step of sixteen uneven bars 13.69 and 11.48 ms.  Launches that
// fill the chip lose nothing, though the gradient then has the element Hessians'
// registers: coloured 81x21x21 patch beam, two iterations, float64 2885 and 2819 us,
// float32 1938 and 1897; 64 patch bars coloured, float64 7.64 and 7.67 ms, float32 4.86
// and 4.78; corotated Jacobi, float64 3.14 and 3.05.
template <typename T, int D, bool FCR>
__device__ __forceinline__ void point_body(const MeshView& mv, int b, const double* __restrict__ x,
                                           const double* __restrict__ xt, const Material& mat, T* __restrict__ est,
                                           const int* elist, int ecount, const int* __restrict__ nptr,
                                           const int* __restrict__ nidx, const double* __restrict__ Xr,
                                           double* __restrict__ rot, double* __restrict__ g) {
  constexpr int TH = elem_threads<T>();
  const int tid = threadIdx.x;
  const int nr = rot != nullptr ? (mv.nf + TH - 1) / TH : 0, ne = (ecount + EWG - 1) / EWG;
  if (b < nr) {
    rotation_body<D>(mv, b * TH + tid, x, nptr, nidx, Xr, rot);
  } else if (b < nr + ne) {
    elem_hess_split<T, D>(mv, (b - nr) * EWG, x, T(mat.mu), T(mat.lam), FCR ? mat.model : MAT_SNH, T(mat.s_el), est,
                          elist, ecount);
  } else if (g != nullptr) {
    (void)gradient_body<D, GRAD_G, FCR>(mv, grad_vertex(mv, (b - nr - ne) * (TH / GRAD_G) + tid / GRAD_G),
                                        tid % GRAD_G, x, xt, mat, g);
  }
}

// Workgroups of point_body for a mesh.
template <typename T>
static int point_blocks(const MeshView& mv, int ecount, bool rot, bool grad) {
  constexpr int TH = elem_threads<T>();
  return (rot ? nblocks(mv.nf, TH) : 0) + nblocks(ecount, EWG) + (grad ? nblocks(mv.nf, TH / GRAD_G) : 0);
}

template <typename T, int D, bool FCR>
__global__ void __launch_bounds__(elem_threads<T>()) k_point(MeshView mv, const double* __restrict__ x,
                                                             const double* __restrict__ xt, Material mat,
                                                             T* __restrict__ est, const int* elist, int ecount,
                                                             const int* __restrict__ nptr,
                                                             const int* __restrict__ nidx,
                                                             const double* __restrict__ Xr,
                                                             double* __restrict__ rot, double* __restrict__ g) {
  point_body<T, D, FCR>(mv, blockIdx.x, x, xt, mat, est, elist, ecount, nptr, nidx, Xr, rot, g);
}

template <typename T, int D, bool FCR>
static void point(const MeshView& mv, const double* x, const double* xt, const Material& mat, void* est,
                  const int* elist, int ecount, const int* nptr, const int* nidx, const double* Xr, double* rot,
                  double* g, hipStream_t s) {
  const int nb = point_blocks<T>(mv, ecount, rot != nullptr, g != nullptr);
  if (nb > 0)
    k_point<T, D, FCR><<<nb, elem_threads<T>(), 0, s>>>(mv, x, xt, mat, (T*)est, elist, ecount, nptr, nidx, Xr, rot,
                                                       g);
}

void launch_point(const MeshView& mv, int prec, const double* x, const double* xt, const Material& mat, void* estore,
                  const int* elist, int ecount, const int* nptr, const int* nidx, const double* Xr, double* rot,
                  double* g, hipStream_t s) {
  if (prec == 0)
    CC_DISPATCH_MAT(mat.model == MAT_FCR, CC_DISPATCH_D(mv.D, point<double, D, FCR>(mv, x, xt, mat, estore, elist,
                                                                                   ecount, nptr, nidx, Xr, rot, g, s)));
  else
    CC_DISPATCH_MAT(mat.model == MAT_FCR, CC_DISPATCH_D(mv.D, point<float, D, FCR>(mv, x, xt, mat, estore, elist,
                                                                                  ecount, nptr, nidx, Xr, rot, g, s)));
}

void launch_energy_grad(const MeshView& mv, const double* x, const double* xt, const Material& mat, double* g,
                        double* partials, int* ne, int* ng, hipStream_t s) {
  const int nbe = nblocks(mv.m, WG);
  *ne = nbe + nblocks(mv.nf, WG);
  *ng = nblocks(mv.nf, WG / GRAD_G);
  if (*ne + *ng == 0) return;
  CC_DISPATCH_MAT(mat.model == MAT_FCR,
                  CC_DISPATCH_D(mv.D, k_energy_grad<D, GRAD_G, FCR><<<*ne + *ng, WG, 0, s>>>(mv, x, xt, mat, nbe,
                                                                                             *ne, g, partials)));
}
void launch_reduce_eg(const double* partials, int ne, int ng, int first, int sums,
                      const unsigned long long* counters, int nc, double* out, hipStream_t s) {
  k_reduce_eg<<<sums, WG, 0, s>>>(partials, ne, ng, first, counters, nc, out);
}
void launch_axpy(int count, const double* x, const double* d, double alpha, double* out,
                 hipStream_t s) {
  if (count <= 0) return;
  k_axpy<<<nblocks(count, WG), WG, 0, s>>>(count, x, d, alpha, out);
}

void launch_probe_element(const MeshView& mv, int prec, const double* x_user, const int* vperm_inv,
                          const int* eperm, double* xi_tmp, const Material& mat, double* ge,
                          double* He, hipStream_t s) {
  (void)x_user;
  (void)vperm_inv;
  // xi_tmp holds internal-order positions; the caller gathered them already.
  // estore scratch follows the positions in the same allocation.
  const int nb = nblocks(mv.m, WG);
  double* est = xi_tmp + (size_t)mv.D * mv.n;
  launch_elem_hess(mv, prec, xi_tmp, mat, 1.0, est, s);
  if (prec == 0)
    CC_DISPATCH_D(mv.D, k_probe_elem<double, D><<<nb, WG, 0, s>>>(mv, xi_tmp, eperm, (const double*)est,
                                                                 mat.mu, mat.lam, mat.model, ge, He));
  else
    CC_DISPATCH_D(mv.D, k_probe_elem<float, D><<<nb, WG, 0, s>>>(mv, xi_tmp, eperm, (const float*)est,
                                                                (float)mat.mu, (float)mat.lam, mat.model, ge,
                                                                He));
}

void launch_gather_user(const MeshView& mv, const int* vperm_inv, const double* src_user,
                        double* dst_int, hipStream_t s) {
  CC_DISPATCH_D(mv.D, k_gather_user<D><<<nblocks(mv.n, WG), WG, 0, s>>>(mv, vperm_inv, src_user, dst_int));
}

void launch_scatter_user(const MeshView& mv, const int* vperm, const double* src_int,
                         double* dst_user, int free_only, hipStream_t s) {
  CC_DISPATCH_D(mv.D, k_scatter_user<D><<<nblocks(mv.n, WG), WG, 0, s>>>(mv, vperm, src_int, dst_user,
                                                                        free_only));
}

}  // namespace cc

// ===========================================================================
// Batched stepping: every launch covers all meshes of a batch; block b of a
// launch belongs to mesh m when boff[m] <= b < boff[m+1].  Meshes whose
// control block is inactive return at once, so a captured sequence of
// launches stays valid while meshes finish at different iterations.
namespace cc {


__device__ __forceinline__ const double* pick(const BatchItem& it, int which) {
  return which ? it.xtrial : it.x;
}

__device__ __forceinline__ void vertex_range(const BatchItem& it, int colour, int& v0, int& v1) {
  if (colour < 0) { v0 = 0; v1 = it.mv.nf; }
  else if (colour < it.ncol) { v0 = it.coff[colour]; v1 = it.coff[colour + 1]; }
  else { v0 = v1 = 0; }
}

// Start of a step: control block and fallback counters of every mesh.
__global__ void kb_reset(const BatchItem* __restrict__ items, BatchCtl* ctl, int nmesh) {
  const int m = blockIdx.x * WG + threadIdx.x;
  if (m >= nmesh) return;
  BatchCtl c{};
  c.active = 1;
  c.status = -100;
  ctl[m] = c;
  unsigned long long* fb = items[m].fb;
#pragma unroll
  for (int q = 0; q < 4; ++q) fb[q] = 0ull;
}

template <int D>
__global__ void __launch_bounds__(WG) kb_predict(const BatchItem* __restrict__ items, BatchCtl* ctl,
                                                 const int* __restrict__ boff, int nmesh, double h,
                                                 int quasi) {
  const int mi = block_mesh(boff, nmesh, blockIdx.x);
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  const int v = (blockIdx.x - boff[mi]) * WG + threadIdx.x;
  if (v >= mv.n) return;
  const int u = mv.vperm[v], n = mv.n;
  bool ok = true;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const double xp = it.xu[u * D + c], vp = it.vu[u * D + c];
    ok = ok && isfinite(xp) && isfinite(vp);
    it.x0[c * n + v] = xp;
    double xh;
    if (v < mv.nf) {
      xh = quasi ? xp : xp + h * vp;
    } else {
      xh = it.xbc ? it.xbc[u * D + c] : xp;
      ok = ok && isfinite(xh);
    }
    it.xt[c * n + v] = xh;
    it.x[c * n + v] = xh;
    // both position buffers start equal, so the Dirichlet entries of the
    // trial buffer hold the targets whichever buffer the step ends in
    it.xtrial[c * n + v] = xh;
  }
  if (!ok) atomicOr(&ctl[mi].bad, 1);
}

template <int D>
__global__ void __launch_bounds__(WG) kb_finalize(const BatchItem* __restrict__ items,
                                                  const int* __restrict__ boff, int nmesh, double h,
                                                  int quasi) {
  const int mi = block_mesh(boff, nmesh, blockIdx.x);
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  const int v = (blockIdx.x - boff[mi]) * WG + threadIdx.x;
  if (v >= mv.n) return;
  const int u = mv.vperm[v], n = mv.n;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const double xn = it.x[c * n + v];
    it.xu[u * D + c] = xn;
    it.vu[u * D + c] = quasi ? 0.0 : (xn - it.x0[c * n + v]) / h;
    if (mv.corr) mv.corr[c * n + v] = v < mv.nf ? xn - it.xt[c * n + v] : 0.0;
  }
}

template <typename T, int D, bool FCR>
__global__ void __launch_bounds__(elem_threads<T>()) kb_elem_hess(const BatchItem* __restrict__ items,
                                                   const BatchCtl* __restrict__ ctl,
                                                   const int* __restrict__ boff, int nmesh, int which,
                                                   int colour) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  // colour >= 0: only the elements that colour's moves changed
  const bool lst = colour >= 0 && colour < it.ncol;
  const int* el = lst ? mv.cel + mv.cel_ptr[colour] : nullptr;
  const int cnt = lst ? mv.cel_ptr[colour + 1] - mv.cel_ptr[colour] : mv.m;
  elem_hess_split<T, D>(mv, (bx - boff[mi]) * EWG, pick(it, which), T(it.mat.mu), T(it.mat.lam),
                        FCR ? it.mat.model : MAT_SNH, T(it.mat.s_el), (T*)it.estore, el, cnt);
}

// point_body of every mesh at positions `which` (grad: with the gradient).
template <typename T, int D, bool FCR>
__global__ void __launch_bounds__(elem_threads<T>()) kb_point(const BatchItem* __restrict__ items,
                                                              const BatchCtl* __restrict__ ctl,
                                                              const int* __restrict__ boff, int nmesh, int which,
                                                              int colour, int grad) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  // colour >= 0: only the elements that colour's moves changed
  const bool lst = colour >= 0 && colour < it.ncol;
  const int* el = lst ? mv.cel + mv.cel_ptr[colour] : nullptr;
  const int cnt = lst ? mv.cel_ptr[colour + 1] - mv.cel_ptr[colour] : mv.m;
  point_body<T, D, FCR>(mv, bx - boff[mi], pick(it, which), it.xt, it.mat, (T*)it.estore, el, cnt, it.nptr, it.nidx,
                        it.Xr, const_cast<double*>(mv.rot), grad ? it.g : nullptr);
}

// Corotation: vertex rotations of every mesh at positions `which`.
template <int D>
__global__ void __launch_bounds__(WG) kb_rotations(const BatchItem* __restrict__ items,
                                                   const BatchCtl* __restrict__ ctl,
                                                   const int* __restrict__ boff, int nmesh, int which) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  if (it.mv.rot == nullptr) return;
  rotation_body<D>(it.mv, (bx - boff[mi]) * WG + threadIdx.x, pick(it, which), it.nptr, it.nidx,
                   it.Xr, const_cast<double*>(it.mv.rot));
}

template <typename T, int D>
__global__ void __launch_bounds__(EWG) kb_assemble(const BatchItem* __restrict__ items,
                                                  const BatchCtl* __restrict__ ctl,
                                                  const int* __restrict__ boff, int nmesh, int colour) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  const bool lst = colour >= 0 && colour < it.ncol;
  const int* sl = lst ? mv.csl + mv.csl_ptr[colour] : nullptr;
  const int cnt = lst ? mv.csl_ptr[colour + 1] - mv.csl_ptr[colour] : mv.nnzb;
  assemble_body<T, D>(mv, (bx - boff[mi]) * EWG + threadIdx.x, (const T*)it.estore,
                      T(it.mat.w_in), (T*)it.hb, mv.tile ? it.g : nullptr, sl, cnt);
}

template <int D, int G, bool FCR>
__global__ void __launch_bounds__(WG) kb_gradient(const BatchItem* __restrict__ items,
                                                  const BatchCtl* __restrict__ ctl,
                                                  const int* __restrict__ boff, int nmesh, int which,
                                                  int only_warm) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  __shared__ double red[WG];
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active || (only_warm && !ctl[mi].warm)) return;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  const int lb = bx - boff[mi];
  const double gsq = gradient_body<D, G, FCR>(mv, grad_vertex(mv, lb * (WG / G) + threadIdx.x / G), threadIdx.x % G,
                                         pick(it, which), it.xt, it.mat, it.g);
  const double tot = block_sum<WG>(gsq, red);
  if (threadIdx.x == 0) it.partials[lb] = tot;
}

template <typename T, int D, int G>
__global__ void __launch_bounds__(WG) kb_prep(const BatchItem* __restrict__ items,
                                              const BatchCtl* __restrict__ ctl,
                                              const int* __restrict__ boff, int nmesh, int method,
                                              int colour, int cap) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  int v0, v1;
  vertex_range(it, colour, v0, v1);
  const int idx = (bx - boff[mi]) * (WG / G) + threadIdx.x / G;
  const bool act = idx < v1 - v0;
  prep_body<T, D, G>(it.mv, method, act ? sweep_vertex(it.mv, v0, v1, idx) : v0, act, threadIdx.x % G,
                     (const T*)it.hb, (T*)it.KL, it.fb,
                     cap > 0 ? reinterpret_cast<T*>(smem_raw) : nullptr, cap);
}

// Dense-basis meshes of a batch: TV vertices per workgroup (prep_band_body).
// Blocks boff[k] .. boff[k + 1] belong to mesh order[k]: the meshes by falling
// nf, since a workgroup's time grows with nf and the launch ends sooner when
// the long workgroups start first.
template <typename T, int D, int TV, int CH>
__global__ void __launch_bounds__(CH) kb_prep_band(const BatchItem* __restrict__ items,
                                                    const BatchCtl* __restrict__ ctl,
                                                    const int* __restrict__ boff,
                                                    const int* __restrict__ order, int nmesh,
                                                    int colour, int fuse, int nseg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int slot = block_mesh(boff, nmesh, blockIdx.x), mi = order[slot];
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  int v0, v1;
  vertex_range(it, colour, v0, v1);
  const int lb = blockIdx.x - boff[slot], nb = (boff[slot + 1] - boff[slot]) / nseg, i0 = v0 + lb % nb * TV;
  prep_band_body<T, D, TV, CH>(it.mv, i0, min(TV, v1 - i0), (const T*)it.hb, (T*)it.KL,
                           reinterpret_cast<T*>(smem_raw), fuse ? it.g : nullptr, fuse ? it.d : nullptr, lb / nb,
                           nseg);
}

template <int NG, int NS, int CH>
__global__ void __launch_bounds__(64 * NS, 4)
kb_prep_tile(const BatchItem* __restrict__ items, const BatchCtl* __restrict__ ctl, const int* __restrict__ boff,
             const int* __restrict__ order, int nmesh, int colour, int fuse, int nseg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int slot = block_mesh(boff, nmesh, blockIdx.x), mi = order[slot];
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  int v0, v1;
  vertex_range(it, colour, v0, v1);
  const int lb = blockIdx.x - boff[slot], nb = (boff[slot + 1] - boff[slot]) / nseg, i0 = v0 + lb % nb * 5 * NG;
  prep_tile_body<NG, NS, CH>(it.mv, i0, min(5 * NG, v1 - i0), (const float*)it.hb, (float*)it.KL,
                             reinterpret_cast<float*>(smem_raw), fuse ? it.d : nullptr, lb / nb, nseg);
}

template <typename T, int D>
__global__ void __launch_bounds__(WG) kb_dm_finish(const BatchItem* __restrict__ items,
                                                   const BatchCtl* __restrict__ ctl,
                                                   const int* __restrict__ boff, int nmesh,
                                                   int method, int colour, int fuse, int nseg,
                                                   const int* __restrict__ segs) {
  const int mi = block_mesh(boff, nmesh, blockIdx.x);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  int v0, v1;
  vertex_range(it, colour, v0, v1);
  const int i = v0 + (blockIdx.x - boff[mi]) * WG + threadIdx.x;
  // fuse 1 (Jacobi): xtrial = x + d; fuse 2 (coloured sweep): the colour's
  // vertices move in place in the sweep's running state xtrial
  if (i < v1)
    dm_finish_body<T, D>(it.mv, method, i, (const T*)it.hb, (T*)it.KL, it.fb, fuse ? it.g : nullptr,
                         fuse ? it.d : nullptr, fuse == 2 ? it.xtrial : it.x, fuse ? it.xtrial : nullptr,
                         segs != nullptr ? segs[mi] : nseg);
}

template <typename T, int D, int G>
__global__ void __launch_bounds__(WG) kb_update(const BatchItem* __restrict__ items,
                                                const BatchCtl* __restrict__ ctl,
                                                const int* __restrict__ boff, int nmesh, int method,
                                                int colour, int into_trial) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  int v0, v1;
  vertex_range(it, colour, v0, v1);
  const int i = v0 + (bx - boff[mi]) * (WG / G) + threadIdx.x / G;
  update_body<T, D, G>(mv, method, i, i < v1, threadIdx.x % G, (const T*)it.KL, it.g,
                       into_trial ? it.xtrial : it.d, into_trial);
}

// xtrial = x + alpha d (copy_only: xtrial = x) over all D*n entries.
__global__ void __launch_bounds__(WG) kb_axpy(const BatchItem* __restrict__ items,
                                              const BatchCtl* __restrict__ ctl,
                                              const int* __restrict__ boff, int nmesh, double alpha,
                                              int copy_only) {
  const int mi = block_mesh(boff, nmesh, blockIdx.x);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const int t = (blockIdx.x - boff[mi]) * WG + threadIdx.x;
  if (t >= it.mv.D * it.mv.n) return;
  it.xtrial[t] = copy_only ? it.x[t] : it.x[t] + alpha * it.d[t];
}

// The end of a line-searched iteration in one launch: per mesh, the energy
// blocks at the trial point (as kb_energy) followed by the gradient blocks
// at the trial point (as kb_gradient), each writing its partial at its own
// block index.  The gradient is speculative: it is used only if the trial
// point is taken, and every path that leaves a mesh at its old x computes
// the gradient there again.
template <int D, bool FCR>
__global__ void __launch_bounds__(WG) kb_energy_grad(const BatchItem* __restrict__ items,
                                                     const BatchCtl* __restrict__ ctl,
                                                     const int* __restrict__ boff, int nmesh) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  __shared__ double red[WG];
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  const int lb = bx - boff[mi];
  const int nbe = (mv.m + WG - 1) / WG;
  const int ne = nbe + (mv.nf + WG - 1) / WG;
  double v;
  if (lb < ne)
    v = energy_body<D, FCR>(mv, lb, nbe, it.xtrial, it.xt, it.mat);
  else
    v = gradient_body<D, GRAD_G, FCR>(mv, grad_vertex(mv, (lb - ne) * (WG / GRAD_G) + threadIdx.x / GRAD_G),
                                      threadIdx.x % GRAD_G, it.xtrial, it.xt, it.mat, it.g);
  const double tot = block_sum<WG>(v, red);
  if (threadIdx.x == 0) it.partials[lb] = tot;
}

template <int D, bool FCR>
__global__ void __launch_bounds__(WG) kb_energy(const BatchItem* __restrict__ items,
                                                const BatchCtl* __restrict__ ctl,
                                                const int* __restrict__ boff, int nmesh, int which) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  __shared__ double red[WG];
  const int mi = block_mesh(boff, nmesh, bx);
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  const int lb = bx - boff[mi];
  const int nbe = (mv.m + WG - 1) / WG;
  const double v = energy_body<D, FCR>(mv, lb, nbe, pick(it, which), it.xt, it.mat);
  const double tot = block_sum<WG>(v, red);
  if (threadIdx.x == 0) it.partials[lb] = tot;
}

// Accept the iteration of an active mesh when E did not rise beyond the
// slack (or without line search); otherwise hand the mesh to the host for
// backtracking.
__device__ __forceinline__ void accept_mesh(BatchItem& item, BatchCtl& c, int line_search) {
  const double tau = 1e-12 * fmax(fabs(c.E_cur), 1.0);
  if (!line_search || c.E_trial <= c.E_cur + tau) {
    double* t = item.x;
    item.x = item.xtrial;
    item.xtrial = t;
    if (line_search) c.E_cur = c.E_trial;
    c.iters += 1;
  } else {
    c.needs_host = 1;
    c.active = 0;
  }
}

// Learned warm start: the proposal (in xtrial, its energy in E_trial)
// replaces the predictor when it has the lower step energy.
// tag: 1 the network's proposal, 2 the previous correction alone
__device__ __forceinline__ void warm_accept_mesh(BatchItem& item, BatchCtl& c, int tag) {
  if (c.E_trial < c.E_cur) {
    double* t = item.x;
    item.x = item.xtrial;
    item.xtrial = t;
    c.E_cur = c.E_trial;
    c.warm = tag;
  }
}

// Residual at an accepted proposal against the predictor's gradient norm g0.
__device__ __forceinline__ void warm_check_mesh(BatchCtl& c, double tol) {
  c.r = sqrt(c.gn2) / c.g0;
  if (c.r <= tol) { c.status = 0; c.active = 0; }
}

// Convergence test of an active mesh after its gradient norm is in gn2.
__device__ __forceinline__ void converged_mesh(BatchCtl& c, double tol, int max_iters) {
  c.r = sqrt(c.gn2) / c.g0;
  if (!isfinite(c.r)) { c.status = 2; c.active = 0; }
  else if (c.r <= tol) { c.status = 0; c.active = 0; }
  else if (c.iters >= max_iters) { c.status = 1; c.active = 0; }
}

// One workgroup per mesh: sums the partials written by the launch whose
// block offsets are boff_src; dst 0 -> E_trial, 1 -> gn2, 2 -> E_cur.  Then,
// on the same thread, post 1 applies the accept rule (dst 0) and post 2 the
// convergence test (dst 1), saving the launch of kb_accept / kb_converged.
// only_warm: meshes whose learned proposal was rejected are skipped (their
// positions, gradient and norm are those of the predictor, already known).
// Sum of a mesh's per-block partials, in a fixed order (the single-mesh
// k_reduce sums the same way).
__device__ __forceinline__ double mesh_partials_sum(const BatchItem& it, int np, double* red) {
  double v = 0.0;
  for (int i = threadIdx.x; i < np; i += WG) v += it.partials[i];
  return block_sum<WG>(v, red);
}

__global__ void __launch_bounds__(WG) kb_reduce(BatchItem* __restrict__ items, BatchCtl* ctl,
                                                const int* __restrict__ boff_src, int dst, int post,
                                                double tol, int max_iters, int only_warm) {
  __shared__ double red[WG];
  const int mi = blockIdx.x;
  if (!ctl[mi].active || (only_warm && !ctl[mi].warm)) return;
  const double tot = mesh_partials_sum(items[mi], boff_src[mi + 1] - boff_src[mi], red);
  if (threadIdx.x == 0) {
    BatchCtl& c = ctl[mi];
    if (dst == 0) c.E_trial = tot;
    else if (dst == 1) c.gn2 = tot;
    else c.E_cur = tot;
    if (post == 1) accept_mesh(items[mi], c, 1);
    else if (post == 2) converged_mesh(c, tol, max_iters);
    else if (post == 3) warm_accept_mesh(items[mi], c, 1);
    else if (post == 5) warm_accept_mesh(items[mi], c, 2);
    else if (post == 4) warm_check_mesh(c, tol);
  }
}

// Backtracking (Results, Subspace Quality: global line search along the
// sweep's displacement) of the active meshes, all meshes per launch.  The
// halvings alpha = 1/2, 1/4, ... are tried LS_WIDTH at a time: one launch
// evaluates E(x + alpha d) for each, and the decision takes the first that
// does not raise E, which is what trying them one after another would take.
// ctl.ls: 0 searching, 3 step found (to be written), 1 taken, 2 halvings
// exhausted.

// mode 0: d = x_trial - x for the active meshes; mode 1: x_trial = x + alpha d
// for the meshes whose step was found.
__global__ void __launch_bounds__(WG) kb_ls_vec(BatchItem* __restrict__ items,
                                                const BatchCtl* __restrict__ ctl,
                                                const int* __restrict__ boff, int nmesh, int mode) {
  const int mi = block_mesh(boff, nmesh, blockIdx.x);
  if (!ctl[mi].active || (mode == 1 && ctl[mi].ls != 3)) return;
  const BatchItem& it = items[mi];
  const int t = (blockIdx.x - boff[mi]) * WG + threadIdx.x;
  if (t >= it.mv.D * it.mv.n) return;
  if (mode == 0) it.d[t] = it.xtrial[t] + -1.0 * it.x[t];
  else it.xtrial[t] = it.x[t] + ctl[mi].alpha * it.d[t];
}

// Energy partials at x + alpha_k d, alpha_k = ctl.alpha / 2^k, k = blockIdx.y,
// laid out as kb_energy's partials, one set of `total` per k.
template <int D, bool FCR>
__global__ void __launch_bounds__(WG) kb_energy_wide(const BatchItem* __restrict__ items,
                                                     const BatchCtl* __restrict__ ctl,
                                                     const int* __restrict__ boff, int nmesh,
                                                     int total, int max_halvings,
                                                     double* __restrict__ wpart) {
  // blocks of one XCD take a contiguous range of the launch (one mesh, or
  // neighbouring ones), so each mesh's data stays in one L2
  const int bx = xcd_block(blockIdx.x, gridDim.x);
  __shared__ double red[WG];
  const int mi = block_mesh(boff, nmesh, bx);
  const BatchCtl& c = ctl[mi];
  const int k = blockIdx.y;
  if (!c.active || c.ls != 0 || c.halvings + k > max_halvings) return;
  double alpha = c.alpha;
  for (int q = 0; q < k; ++q) alpha *= 0.5;
  const BatchItem& it = items[mi];
  const MeshView mv = it.mv;
  const int lb = bx - boff[mi];
  const int nbe = (mv.m + WG - 1) / WG;
  const double v = energy_body_along<D, FCR>(mv, lb, nbe, it.x, it.d, alpha, it.xt, it.mat);
  const double tot = block_sum<WG>(v, red);
  if (threadIdx.x == 0) wpart[(size_t)k * total + bx] = tot;
}

// Per mesh, in halving order: E at alpha_k (partials summed as kb_reduce
// sums them); the first that does not raise E beyond the slack is the step;
// at the halving limit the search stops; otherwise the next launch goes on
// from alpha / 2^width.
__global__ void __launch_bounds__(WG) kb_ls_reduce_wide(BatchCtl* ctl, const int* __restrict__ boff,
                                                        int total, int width, int max_halvings,
                                                        const double* __restrict__ wpart) {
  __shared__ double red[WG];
  const int mi = blockIdx.x;
  BatchCtl& c = ctl[mi];
  if (!c.active || c.ls != 0) return;
  const double tau = 1e-12 * fmax(fabs(c.E_cur), 1.0);
  const double Ecur = c.E_cur;
  const int np = boff[mi + 1] - boff[mi];
  double alpha = c.alpha, Et = 0.0;
  int h = c.halvings, ls = 0;
  for (int k = 0; k < width; ++k) {
    const double* part = wpart + (size_t)k * total + boff[mi];
    double v = 0.0;
    for (int i = threadIdx.x; i < np; i += WG) v += part[i];
    Et = block_sum<WG>(v, red);
    __syncthreads();                       // red is reused by the next sum
    if (Et <= Ecur + tau) { ls = 3; break; }
    if (h >= max_halvings) { ls = 2; break; }
    alpha *= 0.5;
    h += 1;
  }
  if (threadIdx.x != 0) return;
  c.E_trial = Et;
  c.alpha = alpha;
  c.halvings = h;
  c.ls = ls;
  if (ls == 2) c.active = 0;
}

// Takes the written steps: swap x and x_trial, E, one more iteration.
__global__ void kb_ls_commit(BatchItem* __restrict__ items, BatchCtl* ctl, int nmesh) {
  const int mi = blockIdx.x * WG + threadIdx.x;
  if (mi >= nmesh) return;
  BatchCtl& c = ctl[mi];
  if (!c.active || c.ls != 3) return;
  BatchItem& item = items[mi];
  double* t = item.x;
  item.x = item.xtrial;
  item.xtrial = t;
  c.E_cur = c.E_trial;
  c.iters += 1;
  c.ls = 1;
  c.active = 0;
}

// Both sums of kb_energy_grad (each in kb_reduce's order), then the accept
// rule and, for a mesh that took its trial point, the convergence test.
__global__ void __launch_bounds__(WG) kb_reduce_eg(BatchItem* __restrict__ items, BatchCtl* ctl,
                                                   double tol, int max_iters) {
  __shared__ double red[WG];
  const int mi = blockIdx.x;
  if (!ctl[mi].active) return;
  const BatchItem& it = items[mi];
  const int ne = (it.mv.m + WG - 1) / WG + (it.mv.nf + WG - 1) / WG;
  const int ng = (it.mv.nf + WG / GRAD_G - 1) / (WG / GRAD_G);
  const double E = mesh_partials_sum(it, ne, red);
  __syncthreads();                         // red is reused by the next sum
  double v = 0.0;
  for (int i = threadIdx.x; i < ng; i += WG) v += it.partials[ne + i];
  const double gn2 = block_sum<WG>(v, red);
  if (threadIdx.x != 0) return;
  BatchCtl& c = ctl[mi];
  c.E_trial = E;
  accept_mesh(items[mi], c, 1);
  if (c.active) {
    c.gn2 = gn2;
    converged_mesh(c, tol, max_iters);
  }
}

__global__ void kb_init(const BatchItem* items, BatchCtl* ctl, int nmesh, double tol, int max_iters) {
  const int m = blockIdx.x * WG + threadIdx.x;
  if (m >= nmesh) return;
  BatchCtl& c = ctl[m];
  if (c.bad) { c.status = -5; c.active = 0; return; }
  c.g0 = fmax(sqrt(c.gn2), items[m].load);   // relative to the larger of |g(x^0)| and the floor
  if (c.g0 == 0.0) { c.r = 0.0; c.status = 0; c.active = 0; return; }
  c.r = sqrt(c.gn2) / c.g0;
  if (c.r <= tol) { c.status = 0; c.active = 0; }
  else if (max_iters <= 0) { c.status = 1; c.active = 0; }
}

// Accept the iteration when E did not rise beyond the slack (or without line
// search); otherwise hand the mesh to the host for backtracking.
__global__ void kb_accept(BatchItem* items, BatchCtl* ctl, int nmesh, int line_search) {
  const int m = blockIdx.x * WG + threadIdx.x;
  if (m >= nmesh) return;
  if (!ctl[m].active) return;
  accept_mesh(items[m], ctl[m], line_search);
}

// ---- host side of a batch ---------------------------------------------------
struct Offsets {
  std::vector<int> h;
  int* d = nullptr;
  int total() const { return h.empty() ? 0 : h.back(); }
};

// The dense meshes of a batch that share a condensation launch.
struct DenseGroup {
  int tile = 0;     // configuration of the matrix-core condensation (tile_config; 0: the plan's rows of tv)
  size_t lds = 0;   // dynamic LDS of the launch
  std::vector<char> in;       // by mesh
  std::vector<Offsets> prep;  // blocks of the plan's meshes in its order; index 0: all free vertices, c+1: colour c
  std::vector<int> nseg;      // segments of their rows (prep_segments), indexed as prep
};

struct BatchPlan {
  int nmesh = 0;
  BatchConfig cfg{};
  std::vector<BatchItem> items_h;
  BatchItem* items_d = nullptr;
  BatchCtl* ctl_d = nullptr;
  Offsets pred, elem, asmb, grad, energy, axpy, axpyj, feat, rotn;   // axpyj: Jacobi trial points
  Offsets eg;       // energy then gradient blocks of each mesh (kb_energy_grad)
  Offsets point;    // rotations and elements of each mesh (kb_point)
  std::vector<Offsets> pointg;   // with the gradient; index 0: all elements, c + 1: colour c's dirty ones
  std::vector<Offsets> elemc, asmbc;   // element / slot blocks of colour c's dirty lists
  std::vector<Offsets> prep, fin, upd;   // index 0: all free vertices, c+1: colour c
  Offsets fseg;     // with several groups: the segments of every mesh's rows, nmesh for each entry of fin
  std::vector<DenseGroup> dense;         // none: no dense mesh
  std::vector<int> dorder_h;  // meshes by falling nf: the order of the groups' blocks
  int* dorder = nullptr;
  int max_colours = 0;
  int tv = 0;       // vertices per workgroup of the band kernel (0: no dense mesh)
  int ch = 0;       // its chunk of band positions (= workgroup size)
  int scap = 0;     // staged support blocks per vertex of the sparse condensation (0: none)
  size_t slds = 0;  // its dynamic LDS
  double* wpart = nullptr;   // energy partials of LS_WIDTH backtracking steps
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  int graph_iters = 0;
  BatchHook hook = nullptr;
  void* hook_user = nullptr;
  int capturing = 0;
  int capture_failed = 0;   // graph capture failed: the iterations run uncaptured
  void mark(int kid, int begin) { if (hook) hook(hook_user, kid, begin); }
};

static void drop_graph(BatchPlan* p) {
  if (p->exec) { (void)hipGraphExecDestroy(p->exec); p->exec = nullptr; }
  if (p->graph) { (void)hipGraphDestroy(p->graph); p->graph = nullptr; }
}

void batch_set_hook(BatchPlan* p, BatchHook hook, void* user) {
  if (p->hook == hook && p->hook_user == user) return;
  drop_graph(p);
  p->hook = hook;
  p->hook_user = user;
}

int batch_capturing(BatchPlan* p) { return p->capturing; }
int batch_has_graph(BatchPlan* p) { return p->exec != nullptr; }

static void offsets_upload(Offsets& o, hipStream_t s) {
  if (o.d) (void)hipFree(o.d);
  (void)hipMalloc(&o.d, o.h.size() * sizeof(int));
  (void)hipMemcpyAsync(o.d, o.h.data(), o.h.size() * sizeof(int), hipMemcpyHostToDevice, s);
}

static void offsets_build(Offsets& o, const std::vector<int>& counts, hipStream_t s) {
  o.h.assign(counts.size() + 1, 0);
  for (size_t i = 0; i < counts.size(); ++i) o.h[i + 1] = o.h[i] + counts[i];
  offsets_upload(o, s);
}

static void offsets_free(Offsets& o) {
  if (o.d) (void)hipFree(o.d);
  o.d = nullptr;
}

static void vertex_offsets_free(BatchPlan* p) {
  for (auto* v : {&p->prep, &p->fin, &p->upd, &p->elemc, &p->asmbc})
    for (auto& o : *v) offsets_free(o);
  offsets_free(p->fseg);
  for (auto& g : p->dense)
    for (auto& o : g.prep) offsets_free(o);
}

// Blocks of a group's meshes for colour c (cnt: every mesh's vertices of that
// colour), and the segments of their rows, which nseg receives for each mesh.
static void group_offsets(const BatchPlan* p, DenseGroup& g, const std::vector<int>& cnt, std::vector<int>& nseg,
                          hipStream_t s) {
  std::vector<int> blocks(p->nmesh);
  int max_nf = 0, unit = p->ch;                       // the longest of these rows, and its segments' unit
  long long rows = 0;
  for (int k = 0; k < p->nmesh; ++k) {
    const int m = p->dorder_h[k];
    if (!g.in[m]) continue;
    const MeshView& mv = p->items_h[m].mv;
    blocks[k] = nblocks(cnt[m], g.tile > 0 ? 5 * TILE_G[g.tile - 1] : p->tv);
    rows += (long long)blocks[k] * mv.nf;
    if (blocks[k] > 0 && mv.nf > max_nf) {
      max_nf = mv.nf;
      if (g.tile > 0) unit = tile_ring(g.tile, mv.nf, mv.band_w);
    }
  }
  const int resident = g.tile > 0 ? tile_resident(g.tile) : dense_resident(DenseCfg{p->tv, p->ch, g.lds}, p->cfg.prec);
  const int ns = prep_segments(g.tile == 0 && p->cfg.prec == 1, max_nf, rows, unit, resident);
  for (int& b : blocks) b *= ns;
  for (int m = 0; m < p->nmesh; ++m)
    if (g.in[m]) nseg[m] = ns;
  g.nseg.push_back(ns);
  g.prep.emplace_back();
  offsets_build(g.prep.back(), blocks, s);
}

static void plan_vertex_offsets(BatchPlan* p, hipStream_t s) {
  const int G = p->cfg.G;
  p->prep.assign(p->max_colours + 1, Offsets{});
  p->fin.assign(p->max_colours + 1, Offsets{});
  p->fseg.h.clear();
  p->upd.assign(p->max_colours + 1, Offsets{});
  for (auto& g : p->dense) {
    g.prep.clear();
    g.nseg.clear();
  }
  for (int c = -1; c < p->max_colours; ++c) {
    std::vector<int> cnts(p->nmesh), cp(p->nmesh), cf(p->nmesh), cu(p->nmesh), nseg(p->nmesh, 1);
    for (int m = 0; m < p->nmesh; ++m) {
      const BatchItem& it = p->items_h[m];
      int v0, v1;
      if (c < 0) { v0 = 0; v1 = it.mv.nf; }
      else if (c < it.ncol) { v0 = it.coff[c]; v1 = it.coff[c + 1]; }
      else { v0 = v1 = 0; }
      const int cnt = cnts[m] = v1 - v0;
      cp[m] = it.prep_dense ? 0 : nblocks(cnt, WG / G);
      cf[m] = it.prep_dense ? nblocks(cnt, WG) : 0;
      // dense meshes get their direction from the fused condensation: in a
      // Jacobi sweep, and per colour in a coloured sweep with per-colour Hessians
      const bool fused = it.prep_dense && ((c < 0 && p->cfg.sweep == 0) ||
                                           (c >= 0 && p->cfg.sweep == 1 && p->cfg.hess_refresh == 0));
      cu[m] = fused ? 0 : nblocks(cnt, WG / G);
    }
    offsets_build(p->prep[c + 1], cp, s);
    for (auto& g : p->dense) group_offsets(p, g, cnts, nseg, s);
    p->fseg.h.insert(p->fseg.h.end(), nseg.begin(), nseg.end());
    offsets_build(p->fin[c + 1], cf, s);
    offsets_build(p->upd[c + 1], cu, s);
  }
  if (p->dense.size() > 1) offsets_upload(p->fseg, s);
  p->elemc.assign(p->max_colours, Offsets{});
  p->asmbc.assign(p->max_colours, Offsets{});
  for (int c = 0; c < p->max_colours; ++c) {
    std::vector<int> ce(p->nmesh), cs(p->nmesh);
    for (int m = 0; m < p->nmesh; ++m) {
      const BatchItem& it = p->items_h[m];
      ce[m] = c < it.ncol ? nblocks(it.cel_n[c], EWG) : 0;
      cs[m] = c < it.ncol ? nblocks(it.csl_n[c], EWG) : 0;
    }
    offsets_build(p->elemc[c], ce, s);
    offsets_build(p->asmbc[c], cs, s);
  }
}

// Float32 3D meshes with tile records, unless a row count or a chunk is forced:
// the matrix-core condensation takes the plan's dense group over, or parts of it,
// where its launch pays (tile_fills, band_better).
// A launch has one configuration and one LDS size, so meshes whose band leaves
// one workgroup per CU (wide) bring every other mesh of theirs down to that.
// Where the others pay by themselves, each kind has a launch of its own; below
// that a second launch's end costs more than it gives, and the batch takes the
// kernel that the wide meshes prefer.  Steps of five iterations, us, one launch in
// one configuration / this rule / the band kernel for all: a 17x17x17 cube with four
// uneven bars 2445 / 2192 / 2343, with sixteen 6754 / 5220 / 5580, with 64 (four
// iterations) 17200 / 12754 / 13528; three cubes and sixteen bars 8188 / 6606 /
// 6802; a 19x19x19 cube and twelve bars 5280 / 4794 / 6771.
static void tile_groups(BatchPlan* p) {
  if (p->dense.empty()) return;
  const DenseGroup all = p->dense[0];
  const bool by_colour = p->cfg.sweep == 1 && p->cfg.hess_refresh == 0;
  for (int m = 0; m < p->nmesh; ++m)
    if (all.in[m] && !tile_usable(p->items_h[m].mv, p->cfg.prec, p->cfg.tv_cap, p->cfg.chunk)) return;
  auto wide = [&](int m) {
    const MeshView& mv = p->items_h[m].mv;
    return 2 * tile_lds_bytes(3, mv.nf, mv.band_w) > g_lds_limit;
  };
  struct Part {
    DenseGroup g;
    int blocks = 0, band = 0;                         // workgroups of a launch, and of meshes that band_better names
    long long rows = 0, rings = 0;                    // their band rows and ring positions
    bool pays() const { return g.tile > 0 && tile_fills(g.tile, blocks, rows, rings) && 2 * band <= blocks; }
  };
  auto part = [&](auto take) {
    Part r;
    r.g.in.assign(p->nmesh, 0);
    std::vector<int> id, nf, bw, rows;
    for (int m = 0; m < p->nmesh; ++m) {
      if (!all.in[m] || !take(m)) continue;
      const BatchItem& it = p->items_h[m];
      r.g.in[m] = 1;
      id.push_back(m);
      nf.push_back(it.mv.nf);
      bw.push_back(it.mv.band_w);
      rows.push_back(by_colour && it.ncol > 0 ? it.mv.nf / it.ncol : it.mv.nf);
    }
    if (id.empty()) return r;
    r.g.tile = tile_config(nf.data(), bw.data(), rows.data(), (int)id.size());   // > 0: fits each of them
    if (r.g.tile == 0) return r;
    for (size_t k = 0; k < id.size(); ++k) {
      const int b = nblocks(rows[k], 5 * TILE_G[r.g.tile - 1]);
      r.g.lds = std::max(r.g.lds, tile_lds_bytes(r.g.tile, nf[k], bw[k]));
      r.blocks += b;
      r.rows += (long long)b * nf[k];
      r.rings += (long long)b * tile_ring(r.g.tile, nf[k], bw[k]);
      if (band_better(p->items_h[id[k]].mv, r.g.tile, p->cfg.corotate)) r.band += b;
    }
    return r;
  };
  const Part w = part(wide), n = part([&](int m) { return !wide(m); });
  std::vector<Part> parts{w, n};                      // long workgroups first
  if (!n.pays()) {
    if (!w.pays()) return;
    parts = {part([](int) { return true; })};
  }
  p->dense.clear();
  for (const Part& r : parts) {
    if (r.blocks == 0) continue;
    p->dense.push_back(r.g);
    if (parts.size() > 1 && !r.pays()) {
      p->dense.back().tile = 0;
      p->dense.back().lds = all.lds;
    }
  }
  for (const DenseGroup& g : p->dense)
    for (int m = 0; m < p->nmesh; ++m)
      if (g.in[m]) p->items_h[m].mv.tile = g.tile > 0;
}

BatchPlan* batch_plan_create(const BatchItem* items_host, int nmesh, const BatchConfig& cfg,
                             hipStream_t s) {
  BatchPlan* p = new BatchPlan();
  p->nmesh = nmesh;
  p->cfg = cfg;
  p->items_h.assign(items_host, items_host + nmesh);
  std::vector<int> cpred(nmesh), celem(nmesh), casm(nmesh), cgrad(nmesh), cen(nmesh), cax(nmesh),
      caxj(nmesh), cfeat(nmesh), crot(nmesh);
  {
    // one dense configuration (rows per workgroup, chunk, LDS) for every
    // dense-basis mesh; none fitting sends them to the sparse-row kernel
    std::vector<int> dense_nf, dense_bw;
    for (int m = 0; m < nmesh; ++m)
      if (p->items_h[m].prep_dense) {
        dense_nf.push_back(p->items_h[m].mv.nf);
        dense_bw.push_back(p->items_h[m].mv.band_w);
      }
    if (!dense_nf.empty()) {
      // a coloured sweep launches one colour's rows at a time; there chunks of
      // 256 measured faster than the 128 that tie with them on the full mesh
      DenseCfg dc{};
      if (cfg.sweep == 1 && cfg.chunk == 0)
        dc = dense_config(dense_nf.data(), dense_bw.data(), (int)dense_nf.size(), cfg.D, cfg.prec, cfg.tv_cap, 256);
      if (dc.tv == 0)
        dc = dense_config(dense_nf.data(), dense_bw.data(), (int)dense_nf.size(), cfg.D, cfg.prec, cfg.tv_cap,
                          cfg.chunk);
      p->tv = dc.tv;
      p->ch = dc.ch;
      if (dc.tv == 0)
        for (int m = 0; m < nmesh; ++m) p->items_h[m].prep_dense = 0;
      DenseGroup all;
      all.lds = dc.lds;
      all.in.assign(nmesh, 0);
      for (int m = 0; m < nmesh; ++m) all.in[m] = p->items_h[m].prep_dense;
      if (dc.tv > 0) p->dense.push_back(all);
      tile_groups(p);
    }
  }
  int sparse_supp = 0;
  for (int m = 0; m < nmesh; ++m) {
    const MeshView& mv = p->items_h[m].mv;
    cpred[m] = nblocks(mv.n, WG);
    celem[m] = nblocks(mv.m, EWG);
    casm[m] = nblocks(mv.nnzb, EWG);
    cgrad[m] = nblocks(mv.nf, WG / GRAD_G);
    cen[m] = nblocks(mv.m, WG) + nblocks(mv.nf, WG);
    cax[m] = nblocks((long long)mv.D * mv.n, WG);
    // a Jacobi sweep's dense finish writes the trial point itself
    caxj[m] = (cfg.sweep == 0 && p->items_h[m].prep_dense) ? 0 : cax[m];
    cfeat[m] = nblocks(mv.nf, WG / FEAT_LANES);
    crot[m] = (cfg.corotate && mv.rot) ? nblocks(mv.nf, WG) : 0;
    p->max_colours = std::max(p->max_colours, p->items_h[m].ncol);
    if (!p->items_h[m].prep_dense && mv.smap) sparse_supp = std::max(sparse_supp, mv.smap_supp);
  }
  p->scap = sparse_stage_cap(sparse_supp, cfg.G, cfg.D, cfg.prec);
  p->slds = sparse_stage_bytes(p->scap, cfg.G, cfg.D, cfg.prec);

  offsets_build(p->pred, cpred, s);
  offsets_build(p->elem, celem, s);
  offsets_build(p->asmb, casm, s);
  offsets_build(p->grad, cgrad, s);
  offsets_build(p->energy, cen, s);
  {
    std::vector<int> ceg(nmesh);
    for (int m = 0; m < nmesh; ++m) ceg[m] = cen[m] + cgrad[m];
    offsets_build(p->eg, ceg, s);
  }
  if (p->energy.total() > 0 &&
      hipMalloc(&p->wpart, (size_t)LS_WIDTH * p->energy.total() * sizeof(double)) != hipSuccess) {
    (void)hipGetLastError();
    p->wpart = nullptr;
  }
  offsets_build(p->axpy, cax, s);
  offsets_build(p->axpyj, caxj, s);
  offsets_build(p->feat, cfeat, s);
  offsets_build(p->rotn, crot, s);
  // c = -2: without the gradient, -1: with it, all elements
  for (int c = -2; c < (cfg.sweep == 1 ? p->max_colours : -1); ++c) {
    std::vector<int> cp(nmesh);
    for (int m = 0; m < nmesh; ++m) {
      const BatchItem& it = p->items_h[m];
      if (c >= it.ncol && c >= 0) continue;           // the mesh has no such colour
      const int cnt = c >= 0 ? it.cel_n[c] : it.mv.m;
      cp[m] = cfg.prec == 0 ? point_blocks<double>(it.mv, cnt, crot[m] > 0, c > -2)
                            : point_blocks<float>(it.mv, cnt, crot[m] > 0, c > -2);
    }
    if (c > -2) p->pointg.emplace_back();
    offsets_build(c == -2 ? p->point : p->pointg.back(), cp, s);
  }
  p->dorder_h.resize(nmesh);
  for (int m = 0; m < nmesh; ++m) p->dorder_h[m] = m;
  std::stable_sort(p->dorder_h.begin(), p->dorder_h.end(),
                   [&](int a, int b) { return p->items_h[a].mv.nf > p->items_h[b].mv.nf; });
  (void)hipMalloc(&p->dorder, nmesh * sizeof(int));
  (void)hipMemcpyAsync(p->dorder, p->dorder_h.data(), nmesh * sizeof(int), hipMemcpyHostToDevice, s);
  plan_vertex_offsets(p, s);
  (void)hipMalloc(&p->items_d, nmesh * sizeof(BatchItem));
  (void)hipMalloc(&p->ctl_d, nmesh * sizeof(BatchCtl));
  (void)hipMemcpyAsync(p->items_d, p->items_h.data(), nmesh * sizeof(BatchItem), hipMemcpyHostToDevice, s);
  (void)hipStreamSynchronize(s);
  return p;
}

void batch_plan_destroy(BatchPlan* p) {
  if (!p) return;
  drop_graph(p);
  for (Offsets* o : {&p->pred, &p->elem, &p->asmb, &p->grad, &p->energy, &p->eg, &p->axpy, &p->axpyj, &p->feat,
                     &p->rotn, &p->point})
    offsets_free(*o);
  for (auto& o : p->pointg) offsets_free(o);
  vertex_offsets_free(p);
  if (p->dorder) (void)hipFree(p->dorder);
  if (p->wpart) (void)hipFree(p->wpart);
  if (p->items_d) (void)hipFree(p->items_d);
  if (p->ctl_d) (void)hipFree(p->ctl_d);
  delete p;
}

int batch_tile(BatchPlan* p, int m) { return p->items_h[m].mv.tile; }
BatchItem* batch_items_dev(BatchPlan* p) { return p->items_d; }
BatchCtl* batch_ctl_dev(BatchPlan* p) { return p->ctl_d; }

static inline int gridn(const Offsets& o) { return o.total(); }

template <int D>
static void b_gradient(BatchPlan* p, int which, hipStream_t s, int post = 0, int only_warm = 0) {
  if (gridn(p->grad) == 0) return;
  p->mark(2, 1);
  CC_DISPATCH_MAT(p->cfg.any_fcr, kb_gradient<D, GRAD_G, FCR><<<gridn(p->grad), WG, 0, s>>>(
                                      p->items_d, p->ctl_d, p->grad.d, p->nmesh, which, only_warm));
  p->mark(2, 0);
  kb_reduce<<<p->nmesh, WG, 0, s>>>(p->items_d, p->ctl_d, p->grad.d, 1, post, p->cfg.tol,
                                    p->cfg.max_iters, only_warm);
}

template <int D>
static void b_energy(BatchPlan* p, int which, int dst, hipStream_t s, int post = 0) {
  if (gridn(p->energy) == 0) return;
  p->mark(5, 1);
  CC_DISPATCH_MAT(p->cfg.any_fcr, kb_energy<D, FCR><<<gridn(p->energy), WG, 0, s>>>(
                                      p->items_d, p->ctl_d, p->energy.d, p->nmesh, which));
  p->mark(5, 0);
  kb_reduce<<<p->nmesh, WG, 0, s>>>(p->items_d, p->ctl_d, p->energy.d, dst, post, p->cfg.tol,
                                    p->cfg.max_iters, 0);
}

// The gradient at positions `which`, without its norm.
template <int D>
static void b_gradient_only(BatchPlan* p, int which, hipStream_t s) {
  if (gridn(p->grad) == 0) return;
  p->mark(2, 1);
  CC_DISPATCH_MAT(p->cfg.any_fcr, kb_gradient<D, GRAD_G, FCR><<<gridn(p->grad), WG, 0, s>>>(
                                      p->items_d, p->ctl_d, p->grad.d, p->nmesh, which, 0));
  p->mark(2, 0);
}

template <typename T, int D, int G>
static void b_prep(BatchPlan* p, int colour, hipStream_t s, int fuse = 0) {
  const Offsets& o = p->prep[colour + 1];
  const Offsets& of = p->fin[colour + 1];
  if (gridn(o) == 0 && gridn(of) == 0) return;
  p->mark(3, 1);
  if (gridn(o) > 0)
    kb_prep<T, D, G><<<gridn(o), WG, p->slds, s>>>(p->items_d, p->ctl_d, o.d, p->nmesh, p->cfg.method,
                                                  colour, p->scap);
  for (const DenseGroup& g : p->dense) {
    const Offsets& od = g.prep[colour + 1];
    const int nseg = g.nseg[colour + 1];
    if (gridn(od) == 0) continue;
    if (g.tile > 0) {
      CC_DISPATCH_TILE(g.tile, kb_prep_tile<NG, NS, CH><<<gridn(od), 64 * NS, g.lds, s>>>(
                                   p->items_d, p->ctl_d, od.d, p->dorder, p->nmesh, colour, fuse, nseg));
    } else {
      CC_DISPATCH_TVCH(p->tv, p->ch, kb_prep_band<T, D, TV, CH><<<gridn(od), CH, g.lds, s>>>(
                                p->items_d, p->ctl_d, od.d, p->dorder, p->nmesh, colour, fuse, nseg));
    }
  }
  if (gridn(of) > 0)
    kb_dm_finish<T, D><<<gridn(of), WG, 0, s>>>(p->items_d, p->ctl_d, of.d, p->nmesh, p->cfg.method,
                                               colour, fuse, p->dense[0].nseg[colour + 1],
                                               p->dense.size() > 1 ? p->fseg.d + (colour + 1) * p->nmesh : nullptr);
  p->mark(3, 0);
}

template <typename T, int D, int G>
static void b_update(BatchPlan* p, int colour, int into_trial, hipStream_t s) {
  const Offsets& o = p->upd[colour + 1];
  if (gridn(o) == 0) return;
  p->mark(4, 1);
  kb_update<T, D, G><<<gridn(o), WG, 0, s>>>(p->items_d, p->ctl_d, o.d, p->nmesh, p->cfg.method, colour,
                                             into_trial);
  p->mark(4, 0);
}

// Element Hessians and block rows at positions `which`, with the rotations of
// corotated meshes and (grad) the gradient at the same positions: of every
// element (colour < 0), or only those that colour's moves changed.  The
// kernels are launched one by one where they are timed one by one, and where
// only element Hessians are wanted.
template <typename T, int D>
static void b_hessian(BatchPlan* p, int which, hipStream_t s, int colour = -1, bool grad = false) {
  const bool rot = gridn(p->rotn) > 0;
  // band records carry both vertices' rotations, which change everywhere:
  // with them a colour's assembly takes every block too (sixteen uneven bars:
  // 19 us, against 18 for the changed blocks and 7 for the other records)
  const int ac = rot && p->tv > 0 ? -1 : colour;
  const Offsets& oe = colour < 0 ? p->elem : p->elemc[colour];
  const Offsets& oa = ac < 0 ? p->asmb : p->asmbc[ac];
  if (p->hook == nullptr && (rot || grad)) {
    const Offsets& o = grad ? p->pointg[colour + 1] : p->point;
    if (gridn(o) > 0)
      CC_DISPATCH_MAT(p->cfg.any_fcr, kb_point<T, D, FCR><<<gridn(o), elem_threads<T>(), 0, s>>>(
                                          p->items_d, p->ctl_d, o.d, p->nmesh, which, colour, grad));
  } else {
    if (grad) b_gradient_only<D>(p, which, s);
    if (rot) kb_rotations<D><<<gridn(p->rotn), WG, 0, s>>>(p->items_d, p->ctl_d, p->rotn.d, p->nmesh, which);
    if (gridn(oe) > 0) {
      p->mark(0, 1);
      CC_DISPATCH_MAT(p->cfg.any_fcr, kb_elem_hess<T, D, FCR><<<gridn(oe), elem_threads<T>(), 0, s>>>(
                                          p->items_d, p->ctl_d, oe.d, p->nmesh, which, colour));
      p->mark(0, 0);
    }
  }
  if (gridn(oa) > 0) {
    p->mark(1, 1);
    kb_assemble<T, D><<<gridn(oa), EWG, 0, s>>>(p->items_d, p->ctl_d, oa.d, p->nmesh, ac);
    p->mark(1, 0);
  }
}

template <typename T, int D, int G>
static void b_iteration(BatchPlan* p, hipStream_t s) {
  const BatchConfig& c = p->cfg;
  const int nm = p->nmesh, gb = nblocks(nm, WG);
  if (c.sweep == 0) {
    // g holds the gradient at x (from batch_begin or the end of the previous
    // iteration), so the dense condensation forms the direction itself
    b_hessian<T, D>(p, 0, s);
    b_prep<T, D, G>(p, -1, s, 1);
    b_update<T, D, G>(p, -1, 0, s);
    if (gridn(p->axpyj) > 0)
      kb_axpy<<<gridn(p->axpyj), WG, 0, s>>>(p->items_d, p->ctl_d, p->axpyj.d, nm, 1.0, 0);
  } else {
    if (gridn(p->axpy) > 0)
      kb_axpy<<<gridn(p->axpy), WG, 0, s>>>(p->items_d, p->ctl_d, p->axpy.d, nm, 0.0, 1);
    for (int col = 0; col < p->max_colours; ++col) {
      // per-colour Hessians: all of them at the sweep's start, then only the
      // elements and block slots the previous colour's moves changed
      if (c.hess_refresh != 0 && col == 0) {
        b_hessian<T, D>(p, 1, s);
        b_prep<T, D, G>(p, -1, s);
      }
      // dense meshes form b_i from the fresh gradient (which the assembly
      // stores with tile records) and move the colour's vertices in the finish
      // kernel; sparse ones take the update kernel
      if (c.hess_refresh == 0) {
        b_hessian<T, D>(p, 1, s, col == 0 ? -1 : col - 1, true);
        b_prep<T, D, G>(p, col, s, 2);
      } else {
        b_gradient_only<D>(p, 1, s);
      }
      b_update<T, D, G>(p, col, 1, s);
    }
  }
  if (c.line_search) {
    // E and the gradient at the trial point, then the accept rule and the
    // convergence test
    if (gridn(p->eg) > 0) {
      p->mark(5, 1);
      CC_DISPATCH_MAT(c.any_fcr, kb_energy_grad<D, FCR><<<gridn(p->eg), WG, 0, s>>>(
                                     p->items_d, p->ctl_d, p->eg.d, nm));
      p->mark(5, 0);
      kb_reduce_eg<<<nm, WG, 0, s>>>(p->items_d, p->ctl_d, c.tol, c.max_iters);
    }
  } else {
    kb_accept<<<gb, WG, 0, s>>>(p->items_d, p->ctl_d, nm, 0);
    b_gradient<D>(p, 0, s, 2);    // gradient at the accepted point, then the convergence test
  }
}


static void one_iteration(BatchPlan* p, hipStream_t s) {
#define ITER(T, D, G) b_iteration<T, D, G>(p, s)
  const BatchConfig& c = p->cfg;
  if (c.prec == 0) {
    if (c.D == 2) { if (c.G == 64) ITER(double, 2, 64); else if (c.G == 32) ITER(double, 2, 32); else ITER(double, 2, 16); }
    else { if (c.G == 64) ITER(double, 3, 64); else if (c.G == 32) ITER(double, 3, 32); else ITER(double, 3, 16); }
  } else {
    if (c.D == 2) { if (c.G == 64) ITER(float, 2, 64); else if (c.G == 32) ITER(float, 2, 32); else ITER(float, 2, 16); }
    else { if (c.G == 64) ITER(float, 3, 64); else if (c.G == 32) ITER(float, 3, 32); else ITER(float, 3, 16); }
  }
#undef ITER
}

void batch_begin(BatchPlan* p, hipStream_t s) {
  const int nm = p->nmesh, gb = nblocks(nm, WG);
  kb_reset<<<gb, WG, 0, s>>>(p->items_d, p->ctl_d, nm);
  const int D = p->cfg.D;
  if (D == 2) kb_predict<2><<<gridn(p->pred), WG, 0, s>>>(p->items_d, p->ctl_d, p->pred.d, nm, p->cfg.h, p->cfg.quasistatic);
  else kb_predict<3><<<gridn(p->pred), WG, 0, s>>>(p->items_d, p->ctl_d, p->pred.d, nm, p->cfg.h, p->cfg.quasistatic);
  if (D == 2) b_gradient<2>(p, 0, s); else b_gradient<3>(p, 0, s);
  kb_init<<<gb, WG, 0, s>>>(p->items_d, p->ctl_d, nm, p->cfg.tol, p->cfg.max_iters);
  if (p->cfg.line_search) {
    if (D == 2) b_energy<2>(p, 0, 2, s); else b_energy<3>(p, 0, 2, s);
  }
}

hipError_t batch_iterate(BatchPlan* p, int iters, hipStream_t s) {
  const int k = p->cfg.iters_per_graph;
  // with a timing hook the launches run uncaptured: event pairs recorded as
  // graph nodes do not give per-launch durations
  if (k <= 0 || p->hook) {
    for (int i = 0; i < iters; ++i) one_iteration(p, s);
    return hipGetLastError();
  }
  if (!p->exec) {
    bool ok = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) == hipSuccess;
    if (ok) {
      p->capturing = 1;
      for (int i = 0; i < k; ++i) one_iteration(p, s);
      p->capturing = 0;
      ok = hipStreamEndCapture(s, &p->graph) == hipSuccess;
    }
    if (ok) ok = hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0) == hipSuccess;
    if (!ok) {  // capture unsupported on this stream: run the launches directly (reported)
      (void)hipGetLastError();
      if (p->graph) { (void)hipGraphDestroy(p->graph); p->graph = nullptr; }
      p->exec = nullptr;
      p->cfg.iters_per_graph = 0;
      p->capture_failed = 1;
      for (int i = 0; i < iters; ++i) one_iteration(p, s);
      return hipGetLastError();
    }
  }
  for (int done = 0; done < iters; done += k) {
    const hipError_t e = hipGraphLaunch(p->exec, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

int batch_capture_failed(BatchPlan* p) { return p->capture_failed; }

// Pieces of the batched path used by the warm start (cc_mlp.hip).
void batch_energy_trial(BatchPlan* p, hipStream_t s, int post) {
  if (p->cfg.D == 3) b_energy<3>(p, 1, 0, s, post); else b_energy<2>(p, 1, 0, s, post);
}
void batch_gradient_x(BatchPlan* p, hipStream_t s, int only_warm, int post) {
  if (p->cfg.D == 3) b_gradient<3>(p, 0, s, post, only_warm);
  else b_gradient<2>(p, 0, s, post, only_warm);
}
void batch_elem_hess_x(BatchPlan* p, hipStream_t s) {
  const Offsets& oe = p->elem;
  if (gridn(oe) == 0) return;
  if (p->cfg.prec == 0)
    CC_DISPATCH_MAT(p->cfg.any_fcr, kb_elem_hess<double, 3, FCR><<<gridn(oe), elem_threads<double>(), 0, s>>>(
                                        p->items_d, p->ctl_d, oe.d, p->nmesh, 0, -1));
  else
    CC_DISPATCH_MAT(p->cfg.any_fcr, kb_elem_hess<float, 3, FCR><<<gridn(oe), elem_threads<float>(), 0, s>>>(
                                        p->items_d, p->ctl_d, oe.d, p->nmesh, 0, -1));
}
void batch_energy_x(BatchPlan* p, hipStream_t s) {
  if (p->cfg.D == 3) b_energy<3>(p, 0, 2, s); else b_energy<2>(p, 0, 2, s);
}
bool batch_ls_round(BatchPlan* p, int first, int max_halvings, hipStream_t s) {
  const int total = gridn(p->energy);
  if (gridn(p->axpy) == 0 || total == 0) return true;
  if (!p->wpart) return false;
  if (first) kb_ls_vec<<<gridn(p->axpy), WG, 0, s>>>(p->items_d, p->ctl_d, p->axpy.d, p->nmesh, 0);
  const dim3 grid(total, LS_WIDTH);
  p->mark(5, 1);
  if (p->cfg.D == 3)
    CC_DISPATCH_MAT(p->cfg.any_fcr, kb_energy_wide<3, FCR><<<grid, WG, 0, s>>>(
                                        p->items_d, p->ctl_d, p->energy.d, p->nmesh, total,
                                        max_halvings, p->wpart));
  else
    CC_DISPATCH_MAT(p->cfg.any_fcr, kb_energy_wide<2, FCR><<<grid, WG, 0, s>>>(
                                        p->items_d, p->ctl_d, p->energy.d, p->nmesh, total,
                                        max_halvings, p->wpart));
  p->mark(5, 0);
  kb_ls_reduce_wide<<<p->nmesh, WG, 0, s>>>(p->ctl_d, p->energy.d, total, LS_WIDTH, max_halvings,
                                            p->wpart);
  kb_ls_vec<<<gridn(p->axpy), WG, 0, s>>>(p->items_d, p->ctl_d, p->axpy.d, p->nmesh, 1);
  kb_ls_commit<<<(p->nmesh + WG - 1) / WG, WG, 0, s>>>(p->items_d, p->ctl_d, p->nmesh);
  return true;
}

void batch_gradient_converge(BatchPlan* p, hipStream_t s) {
  if (p->cfg.D == 3) b_gradient<3>(p, 0, s, 2); else b_gradient<2>(p, 0, s, 2);
}

BatchGrid batch_grid(BatchPlan* p) {
  BatchGrid g;
  g.nmesh = p->nmesh;
  g.pred_blocks = gridn(p->pred);
  g.pred_off = p->pred.d;
  g.feat_blocks = gridn(p->feat);
  g.feat_off = p->feat.d;
  g.tol = p->cfg.tol;
  g.max_iters = p->cfg.max_iters;
  g.any_fcr = p->cfg.any_fcr;
  g.line_search = p->cfg.line_search;
  g.prec = p->cfg.prec;
  return g;
}

void batch_finish(BatchPlan* p, hipStream_t s) {
  if (gridn(p->pred) == 0) return;
  if (p->cfg.D == 2) kb_finalize<2><<<gridn(p->pred), WG, 0, s>>>(p->items_d, p->pred.d, p->nmesh, p->cfg.h, p->cfg.quasistatic);
  else kb_finalize<3><<<gridn(p->pred), WG, 0, s>>>(p->items_d, p->pred.d, p->nmesh, p->cfg.h, p->cfg.quasistatic);
}

void batch_set_lanes(BatchPlan* p, int G) {
  if (G == p->cfg.G) return;
  p->cfg.G = G;
  drop_graph(p);
  vertex_offsets_free(p);
  plan_vertex_offsets(p, nullptr);
  (void)hipDeviceSynchronize();
}

// Times condensation + update (Jacobi form, writing d only) for lane count G.
float batch_time_prep_update(BatchPlan* p, int G, int reps, hipStream_t s) {
  batch_set_lanes(p, G);
  hipEvent_t a, b;
  (void)hipEventCreate(&a);
  (void)hipEventCreate(&b);
#define PU(T, D, GG) do { b_prep<T, D, GG>(p, -1, s, p->cfg.sweep == 0); b_update<T, D, GG>(p, -1, 0, s); } while (0)
  auto run = [&]() {
    const BatchConfig& c = p->cfg;
    if (c.prec == 0) {
      if (c.D == 2) { if (G == 64) PU(double, 2, 64); else if (G == 32) PU(double, 2, 32); else PU(double, 2, 16); }
      else { if (G == 64) PU(double, 3, 64); else if (G == 32) PU(double, 3, 32); else PU(double, 3, 16); }
    } else {
      if (c.D == 2) { if (G == 64) PU(float, 2, 64); else if (G == 32) PU(float, 2, 32); else PU(float, 2, 16); }
      else { if (G == 64) PU(float, 3, 64); else if (G == 32) PU(float, 3, 32); else PU(float, 3, 16); }
    }
  };
#undef PU
  run();
  (void)hipEventRecord(a, s);
  for (int r = 0; r < reps; ++r) run();
  (void)hipEventRecord(b, s);
  (void)hipEventSynchronize(b);
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, a, b);
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  return ms / reps;
}

}  // namespace cc
