// Exact perturbation basis on the GPU.
//
// With Z = H^{-1} (H the step Hessian over free DOFs), the basis of vertex i
// is U_i[j] = Z_ji Z_ii^{-1}: [I; U_i] spans the columns of Z belonging to
// vertex i, which is U_i = -H_CC^{-1} H_Ci (Method, Coordinate Condensation;
// Background, JGS2).
//
// In band order (breadth-first levels, MeshView::bvert) H is block
// tridiagonal: a block (j, k) couples vertices of the same or of adjacent
// levels.  With D_l = H_ll and B_l = H_{l,l-1} the block LDL^T factorisation
//   S_0 = D_0,  F_l = B_l S_{l-1}^{-1},  S_l = D_l - F_l B_l^T
// gives H = L diag(S) L^T with L unit lower block bidiagonal (L_{l,l-1} = F_l).
// The columns of Z that belong to level q (a "panel") then follow from
//   forward:   Y_q = I,  Y_l = -F_l Y_{l-1}            (l > q; zero above q)
//   diagonal:  Z_l = S_l^{-1} Y_l                        (l >= q)
//   backward:  X_l = Z_l - F_{l+1}^T X_{l+1}             (every l, Z_l = 0 above q)
// and X is column block q of Z = H^{-1}, from which the basis rows of level
// q's vertices are formed directly.  The cost is O(N^2 n) for levels of n
// DOFs instead of the O(N^3) of a dense inverse, the memory O(N n) besides
// the basis itself.  S_l^{-1} comes from a blocked Gauss-Jordan
// inversion (SPD, so its diagonal pivot blocks need no pivoting):
//
//   for every 64-wide block K:  P = A_KK^{-1};  R = P A_K*, P in column K;
//                               C = A_*K;  A_IJ -= C_I R_J (I, J != K);
//                               A_IK = -C_I P;  A_KJ = R_J;  A_KK = P.
//
// Dense matrices are row-major float64.

#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <vector>

#include "cc_device.h"

namespace cc {

constexpr int GJ_B = 64;   // pivot block width
typedef double dbl4 __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and
// C[4 i + l / 16][l % 16], i = 0..3.
__device__ __forceinline__ dbl4 mfma64(double a, double b, dbl4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// P = D^{-1} by Gauss-Jordan for a b x b block, b <= 64, held as a 4 x 4 piece
// m per thread (rows 4 (tid / 16) .., columns 4 (tid % 16) ..; zero past b),
// written to Pout (b x b).  A step passes the pivot's row and column through
// LDS, twice buffered, so that it takes one barrier; a serial chain of b steps
// (about 21 us for b = 64; the block in LDS with five barriers a step took
// 174 us).  row, col: [2][GJ_B] each.
__device__ __forceinline__ void gj_invert(double (&m)[4][4], int b, double (*row)[GJ_B], double (*col)[GJ_B],
                                          double* __restrict__ Pout, int* __restrict__ bad) {
  const int tr = threadIdx.x / 16, tc = threadIdx.x % 16;
  for (int p4 = 0; 4 * p4 < b; ++p4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = 4 * p4 + i;
      if (p >= b) break;                             // uniform
      double *rb = row[i & 1], *cb = col[i & 1];
      if (tr == p4)
#pragma unroll
        for (int w = 0; w < 4; ++w) rb[4 * tc + w] = m[i][w];
      if (tc == p4)
#pragma unroll
        for (int u = 0; u < 4; ++u) cb[4 * tr + u] = m[u][i];
      __syncthreads();
      double piv = rb[p];
      if (!(piv > 0.0)) {
        if (threadIdx.x == 0) atomicOr(bad, 1);
        piv = 1.0;
      }
      // reciprocal by two Newton steps (to about 1 ulp): shorter than the division's chain
      double ip = __builtin_amdgcn_rcp(piv);
      ip = fma(ip, fma(-piv, ip, 1.0), ip);
      ip = fma(ip, fma(-piv, ip, 1.0), ip);
      double rv[4], cv[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) rv[w] = rb[4 * tc + w] * ip;
#pragma unroll
      for (int u = 0; u < 4; ++u) cv[u] = cb[4 * tr + u];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) m[u][w] -= cv[u] * rv[w];
      if (tr == p4)                                  // the pivot's row and column
#pragma unroll
        for (int w = 0; w < 4; ++w) m[i][w] = rv[w];
      if (tc == p4)
#pragma unroll
        for (int u = 0; u < 4; ++u) m[u][i] = tr == p4 && u == i ? ip : -cv[u] * ip;
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int r = 4 * tr + u, c = 4 * tc + w;
      if (r < b && c < b) Pout[r * b + c] = m[u][w];
    }
}

// The first pivot block's inverse.
__global__ void __launch_bounds__(WG) k_gj_first(const double* __restrict__ A, int N, int b,
                                                 double* __restrict__ Pout, int* __restrict__ bad) {
  __shared__ double row[2][GJ_B], col[2][GJ_B];
  const int tr = threadIdx.x / 16, tc = threadIdx.x % 16;
  double m[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int r = 4 * tr + u, c = 4 * tc + w;
      m[u][w] = r < b && c < b ? A[(size_t)r * N + c] : 0.0;
    }
  gj_invert(m, b, row, col, Pout, bad);
}

// One pivot step out of place, 64 x 64 outputs per workgroup: with C = A_*K
// and R = P A_K* (P itself in the pivot's columns),
//   out_IJ = A_IJ - C_I R_J, without A_IJ in the pivot's columns; out_KJ = R_J.
// Every workgroup forms its columns of R itself (half of its products), so the
// whole step is one launch, every element is written once and nothing is read
// that another workgroup writes.  Both products on the float64 matrix cores.
// The workgroup of the next pivot block (launched first) goes on to invert it
// (Pnext): that serial chain is the step's length, the other workgroups run
// beside it.  A step at 780 unknowns: 36 us (about 21 of them the chain); as pivot,
// row, update and column kernels with 4 x 4 outputs per thread it took 230 us.
__global__ void __launch_bounds__(WG) k_gj_step(const double* __restrict__ A, double* __restrict__ out, int N,
                                                int k0, int b, const double* __restrict__ P,
                                                double* __restrict__ Pnext, int* __restrict__ bad) {
  constexpr int T = GJ_B, LC = T + 1, LR = T + 2;    // row strides without bank conflicts
  __shared__ double Cs[T][LC], Rs[T][LR];            // Rs: A_K*, then R
  const int tiles = (N + T - 1) / T, next = k0 / T + 1;
  // tile of this workgroup; the first one and the next pivot's change places
  int t = blockIdx.x;
  const int critical = next < tiles ? next * tiles + next : 0;
  t = t == 0 ? critical : t == critical ? 0 : t;
  const int i0 = t / tiles * T, j0 = t % tiles * T, tid = threadIdx.x, l = tid % 64, w = tid / 64;
  double pf[T / 4];                                  // wave w's rows 16 w .. of P
#pragma unroll
  for (int q = 0; q < T / 4; ++q) {
    const int r = 16 * w + l % 16, k = 4 * q + l / 16;
    const double v = P[min(r, b - 1) * b + min(k, b - 1)];
    pf[q] = r < b && k < b ? v : 0.0;
  }
#pragma unroll
  for (int u = 0; u < T * T / WG; ++u) {
    const int r = (tid + u * WG) / T, q = tid % T;
    const double c = A[(size_t)min(i0 + r, N - 1) * N + min(k0 + q, N - 1)];
    const double a = A[(size_t)min(k0 + r, N - 1) * N + min(j0 + q, N - 1)];
    Cs[r][q] = i0 + r < N && q < b ? c : 0.0;
    Rs[r][q] = r < b && j0 + q < N ? a : 0.0;
  }
  __syncthreads();
  dbl4 acc[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) acc[v] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < T / 4; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = mfma64(pf[q], Rs[4 * q + l / 16][16 * v + l % 16], acc[v]);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 16 * w + 4 * i + l / 16, c = 16 * v + l % 16, kc = j0 + c - k0;
      double x = acc[v][i];
      if (kc >= 0 && kc < b && r < b) x = P[r * b + kc];
      Rs[r][c] = x;
      acc[v][i] = 0.0;
    }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < T / 4; ++q) {
    const double a = Cs[16 * w + l % 16][4 * q + l / 16];
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = mfma64(a, Rs[4 * q + l / 16][16 * v + l % 16], acc[v]);
  }
  const bool invert = next < tiles && i0 == next * T && j0 == next * T;   // uniform
  __syncthreads();                                   // Cs is free
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 16 * w + 4 * i + l / 16, c = 16 * v + l % 16, row = i0 + r, col = j0 + c;
      double x = 0.0;
      if (row < N && col < N) {
        const size_t at = (size_t)row * N + col;
        if (row >= k0 && row < k0 + b) x = Rs[row - k0][c];
        else x = (col >= k0 && col < k0 + b ? 0.0 : A[at]) - acc[v][i];
        out[at] = x;
      }
      if (invert) Cs[r][c] = x;
    }
  if (!invert) return;
  __syncthreads();
  double m[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int x = 0; x < 4; ++x) m[u][x] = Cs[4 * (tid / 16) + u][4 * (tid % 16) + x];
  __syncthreads();
  double(*rowb)[GJ_B] = reinterpret_cast<double(*)[GJ_B]>(&Rs[0][0]);
  gj_invert(m, min(T, N - next * T), rowb, rowb + 2, Pnext, bad);
}

// C (M x N) = alpha op(A) op(B) + beta C, row-major float64, op = transpose
// when TA / TB, on the float64 matrix cores.  A workgroup of four waves forms
// TM x TM outputs, each wave (TM / 2)^2 of them as 16 x 16 tiles; K runs
// through LDS in steps of 16, twice buffered, the next step's loads in flight
// during the products.  With beta = 0, C is not read.  Bound by the matrix
// cores' issue where the tiles fill the chip: 64-wide tiles read less, 32-wide
// ones give four times the workgroups, so they serve outputs of fewer than 256
// of the wide tiles (780 x 780 x 780: 169 wide tiles on 256 CUs).  At that size
// 35 us (27 TFLOP/s); 4 x 4 outputs per thread, an LDS double read for every two
// FMAs, took 157.
constexpr int MM_K = 16;
template <bool TA, bool TB, int TM>
__global__ void __launch_bounds__(WG) k_dgemm(int M, int N, int K, double alpha,
                                              const double* __restrict__ A, int lda,
                                              const double* __restrict__ B, int ldb, double beta,
                                              double* __restrict__ C, int ldc) {
  constexpr int NT = TM / 32, LD = TM + 2, PER = TM * MM_K / WG;   // 16-wide tiles per wave and side; loads
  __shared__ double As[2][MM_K][LD], Bs[2][MM_K][LD];
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TM, tid = threadIdx.x;
  const int l = tid % 64, w = tid / 64, wm = w / 2 * (TM / 2), wn = w % 2 * (TM / 2);
  double va[PER], vb[PER];
  auto load = [&](int kk) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + u * WG;
      // consecutive threads walk the contiguous index of each operand
      const int ma = TA ? e % TM : e / MM_K, ka = TA ? e / TM : e % MM_K;
      const int gm = m0 + ma, gka = kk + ka;
      va[u] = gm < M && gka < K ? (TA ? A[(size_t)gka * lda + gm] : A[(size_t)gm * lda + gka]) : 0.0;
      const int nb = TB ? e / MM_K : e % TM, kb = TB ? e % MM_K : e / TM;
      const int gn = n0 + nb, gkb = kk + kb;
      vb[u] = gn < N && gkb < K ? (TB ? B[(size_t)gn * ldb + gkb] : B[(size_t)gkb * ldb + gn]) : 0.0;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + u * WG;
      As[buf][TA ? e / TM : e % MM_K][TA ? e % TM : e / MM_K] = va[u];
      Bs[buf][TB ? e % MM_K : e / TM][TB ? e / MM_K : e % TM] = vb[u];
    }
  };
  dbl4 acc[NT][NT];
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int v = 0; v < NT; ++v) acc[u][v] = dbl4{0.0, 0.0, 0.0, 0.0};
  load(0);
  store(0);
  __syncthreads();
  for (int kk = 0, buf = 0; kk < K; kk += MM_K, buf ^= 1) {
    const bool more = kk + MM_K < K;
    if (more) load(kk + MM_K);
#pragma unroll
    for (int k4 = 0; k4 < MM_K; k4 += 4) {
      double a[NT], b[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        a[u] = As[buf][k4 + l / 16][wm + 16 * u + l % 16];
        b[u] = Bs[buf][k4 + l / 16][wn + 16 * u + l % 16];
      }
#pragma unroll
      for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int v = 0; v < NT; ++v) acc[u][v] = mfma64(a[u], b[v], acc[u][v]);
    }
    if (more) store(buf ^ 1);                        // read last before the previous barrier
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = m0 + wm + 16 * u + 4 * i + l / 16;
      if (r >= M) continue;
#pragma unroll
      for (int v = 0; v < NT; ++v) {
        const int c = n0 + wn + 16 * v + l % 16;
        if (c >= N) continue;
        double* o = C + (size_t)r * ldc + c;
        const double x = acc[u][v][i];
        *o = beta == 0.0 ? alpha * x : alpha * x + beta * *o;
      }
    }
}

template <bool TA, bool TB>
static void launch_dgemm(int M, int N, int K, double alpha, const double* A, int lda, const double* B, int ldb,
                         double beta, double* C, int ldc, hipStream_t s) {
  auto tiles = [&](int t) { return dim3((N + t - 1) / t, (M + t - 1) / t); };
  const dim3 wide = tiles(64);
  if (wide.x * wide.y >= 256)
    k_dgemm<TA, TB, 64><<<wide, WG, 0, s>>>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
  else
    k_dgemm<TA, TB, 32><<<tiles(32), WG, 0, s>>>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc);
}

static void dgemm(bool ta, bool tb, int M, int N, int K, double alpha, const double* A, int lda,
                  const double* B, int ldb, double beta, double* C, int ldc, hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  if (!ta && !tb) launch_dgemm<false, false>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s);
  else if (!ta && tb) launch_dgemm<false, true>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s);
  else launch_dgemm<true, false>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s);
}

// In-place inverse of the SPD matrix A (N x N); *bad set when a pivot is not
// positive.  tmp: N * N doubles, P: 2 GJ_B^2.  One launch a pivot block.
static void gj_inverse(double* A, int N, double* tmp, double* P, int* bad, hipStream_t s) {
  const int tiles = (N + GJ_B - 1) / GJ_B;
  double *from = A, *to = tmp, *Pk = P, *Pn = P + GJ_B * GJ_B;
  k_gj_first<<<1, WG, 0, s>>>(A, N, std::min(N, GJ_B), Pk, bad);
  for (int k0 = 0; k0 < N; k0 += GJ_B) {
    k_gj_step<<<tiles * tiles, WG, 0, s>>>(from, to, N, k0, std::min(N - k0, GJ_B), Pk, Pn, bad);
    std::swap(from, to);
    std::swap(Pk, Pn);
  }
  if (from != A) (void)hipMemcpyAsync(A, from, (size_t)N * N * sizeof(double), hipMemcpyDeviceToDevice, s);
}

// dst (rows x cols, leading dimension ldd) = alpha src (leading dimension lds)
__global__ void __launch_bounds__(WG) k_scale_copy(double* __restrict__ dst, int ldd,
                                                   const double* __restrict__ src, int lds, int rows,
                                                   int cols, double alpha) {
  const size_t total = (size_t)rows * cols;
  for (size_t e = (size_t)blockIdx.x * WG + threadIdx.x; e < total; e += (size_t)gridDim.x * WG) {
    const size_t r = e / cols, c = e % cols;
    dst[r * ldd + c] = alpha * src[r * lds + c];
  }
}

static void scale_copy(double* dst, int ldd, const double* src, int lds, int rows, int cols, double alpha,
                       hipStream_t s) {
  const size_t total = (size_t)rows * cols;
  if (total == 0) return;
  const int grid = (int)std::min<size_t>((total + WG - 1) / WG, 8192);
  k_scale_copy<<<grid, WG, 0, s>>>(dst, ldd, src, lds, rows, cols, alpha);
}

// Level blocks D_l = H_ll and B_l = H_{l,l-1} from the block rows (both zeroed
// first); lev: level of every band position, loff: first band position of
// every level, oD / oB: offsets of the levels' blocks in Dbuf / Bbuf.
template <int D>
__global__ void k_level_scatter(MeshView mv, const double* __restrict__ hb, const int* __restrict__ lev,
                                const int* __restrict__ loff, const size_t* __restrict__ oD,
                                const size_t* __restrict__ oB, double* __restrict__ Dbuf,
                                double* __restrict__ Bbuf) {
  constexpr int DD = D * D;
  const int t = blockIdx.x * WG + threadIdx.x;
  if (t >= mv.nnzb) return;
  const int pj = mv.bpos[mv.blkrow[t]], pk = mv.bpos[mv.colidx[t]];
  const int lj = lev[pj], lk = lev[pk];
  const int nl = (loff[lj + 1] - loff[lj]) * D;
  double* dst;
  int ld, r0, c0;
  if (lk == lj) {
    dst = Dbuf + oD[lj]; ld = nl; r0 = (pj - loff[lj]) * D; c0 = (pk - loff[lj]) * D;
  } else if (lk == lj - 1) {
    dst = Bbuf + oB[lj]; ld = (loff[lk + 1] - loff[lk]) * D; r0 = (pj - loff[lj]) * D; c0 = (pk - loff[lk]) * D;
  } else {
    return;   // lk == lj + 1: the transpose of B_lk
  }
#pragma unroll
  for (int r = 0; r < D; ++r)
#pragma unroll
    for (int c = 0; c < D; ++c) dst[(size_t)(r0 + r) * ld + c0 + c] = hb[(size_t)t * DD + r * D + c];
}

// Basis rows of the vertices of level q from X = column block q of Z (N x nq,
// rows in band DOF order): U_i[p] = X_p,a X_a,a^{-1} for the level's a-th
// vertex i, zero at its own position.
template <int D>
__global__ void k_basis_from_panel(const double* __restrict__ X, int nq, int q0, int nf,
                                   const int* __restrict__ bvert, double* __restrict__ Ud,
                                   float* __restrict__ Uf) {
  constexpr int DD = D * D;
  const int a = blockIdx.y;
  const int p = blockIdx.x * WG + threadIdx.x;
  if (p >= nf) return;
  const int pa = q0 + a, i = bvert[pa];
  const size_t o = ((size_t)i * nf + p) * DD;
  if (p == pa) {
#pragma unroll
    for (int r = 0; r < DD; ++r) {
      if (Ud) Ud[o + r] = 0.0;
      Uf[o + r] = 0.f;
    }
    return;
  }
  double Zi[D][D], Zinv[D][D];
#pragma unroll
  for (int r = 0; r < D; ++r)
#pragma unroll
    for (int c = 0; c < D; ++c) Zi[r][c] = X[(size_t)(pa * D + r) * nq + a * D + c];
  if constexpr (D == 2) {
    const double det = Zi[0][0] * Zi[1][1] - Zi[0][1] * Zi[1][0];
    Zinv[0][0] = Zi[1][1] / det; Zinv[0][1] = -Zi[0][1] / det;
    Zinv[1][0] = -Zi[1][0] / det; Zinv[1][1] = Zi[0][0] / det;
  } else {
    const double det = Zi[0][0] * (Zi[1][1] * Zi[2][2] - Zi[1][2] * Zi[2][1]) -
                       Zi[0][1] * (Zi[1][0] * Zi[2][2] - Zi[1][2] * Zi[2][0]) +
                       Zi[0][2] * (Zi[1][0] * Zi[2][1] - Zi[1][1] * Zi[2][0]);
    Zinv[0][0] = (Zi[1][1] * Zi[2][2] - Zi[1][2] * Zi[2][1]) / det;
    Zinv[0][1] = (Zi[0][2] * Zi[2][1] - Zi[0][1] * Zi[2][2]) / det;
    Zinv[0][2] = (Zi[0][1] * Zi[1][2] - Zi[0][2] * Zi[1][1]) / det;
    Zinv[1][0] = (Zi[1][2] * Zi[2][0] - Zi[1][0] * Zi[2][2]) / det;
    Zinv[1][1] = (Zi[0][0] * Zi[2][2] - Zi[0][2] * Zi[2][0]) / det;
    Zinv[1][2] = (Zi[0][2] * Zi[1][0] - Zi[0][0] * Zi[1][2]) / det;
    Zinv[2][0] = (Zi[1][0] * Zi[2][1] - Zi[1][1] * Zi[2][0]) / det;
    Zinv[2][1] = (Zi[0][1] * Zi[2][0] - Zi[0][0] * Zi[2][1]) / det;
    Zinv[2][2] = (Zi[0][0] * Zi[1][1] - Zi[0][1] * Zi[1][0]) / det;
  }
#pragma unroll
  for (int r = 0; r < D; ++r)
#pragma unroll
    for (int c = 0; c < D; ++c) {
      double acc = 0.0;
#pragma unroll
      for (int l = 0; l < D; ++l) acc += X[(size_t)(p * D + r) * nq + a * D + l] * Zinv[l][c];
      if (Ud) Ud[o + r * D + c] = acc;
      Uf[o + r * D + c] = (float)acc;
    }
}

bool DeviceScratch::reserve(size_t bytes) {
  if (bytes <= n) return true;
  release();
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    p = nullptr;
    return false;
  }
  n = bytes;
  return true;
}
void DeviceScratch::trim() {
  if (n > KEEP) release();
}
void DeviceScratch::release() {
  if (p) (void)hipFree(p);
  p = nullptr;
  n = 0;
}

int exact_basis_band(const MeshView& mv, const double* hb, const int* loff_h, int L, double* Ud, float* Uf,
                     DeviceScratch& scratch, hipStream_t s) {
  const int D = mv.D, nf = mv.nf, N = nf * D;
  if (nf < 1) return 0;
  std::vector<int> n(L), lev(nf);
  std::vector<size_t> oD(L + 1, 0), oB(L + 1, 0);
  int nmax = 0;
  for (int l = 0; l < L; ++l) {
    n[l] = (loff_h[l + 1] - loff_h[l]) * D;
    nmax = std::max(nmax, n[l]);
    for (int p = loff_h[l]; p < loff_h[l + 1]; ++p) lev[p] = l;
    oD[l + 1] = oD[l] + (size_t)n[l] * n[l];
    oB[l + 1] = oB[l] + (l > 0 ? (size_t)n[l] * n[l - 1] : 0);
  }
  // one workspace for everything, carved in 256-byte steps
  size_t need = 0;
  auto room = [&](size_t bytes) {
    const size_t at = need;
    need += (bytes + 255) / 256 * 256;
    return at;
  };
  const size_t aD = room(oD[L] * 8), aB = room(oB[L] * 8), aT = room((size_t)nmax * nmax * 8),
               aP = room((size_t)N * nmax * 8), aQ = room((size_t)N * nmax * 8), aV = room(2 * GJ_B * GJ_B * 8),
               aoD = room((L + 1) * sizeof(size_t)), aoB = room((L + 1) * sizeof(size_t)),
               alev = room(nf * sizeof(int)), alo = room((L + 1) * sizeof(int)), abad = room(sizeof(int));
  if (!scratch.reserve(need)) return 2;
  char* base = static_cast<char*>(scratch.p);
  double *Dbuf = (double*)(base + aD), *Bbuf = (double*)(base + aB), *tmp = (double*)(base + aT),
         *P = (double*)(base + aP), *Q = (double*)(base + aQ), *pivot = (double*)(base + aV);
  size_t *oD_d = (size_t*)(base + aoD), *oB_d = (size_t*)(base + aoB);
  int *lev_d = (int*)(base + alev), *loff_d = (int*)(base + alo), *bad = (int*)(base + abad);
  auto release = [&]() { scratch.trim(); };
  (void)hipMemcpyAsync(oD_d, oD.data(), (L + 1) * sizeof(size_t), hipMemcpyHostToDevice, s);
  (void)hipMemcpyAsync(oB_d, oB.data(), (L + 1) * sizeof(size_t), hipMemcpyHostToDevice, s);
  (void)hipMemcpyAsync(lev_d, lev.data(), nf * sizeof(int), hipMemcpyHostToDevice, s);
  (void)hipMemcpyAsync(loff_d, loff_h, (L + 1) * sizeof(int), hipMemcpyHostToDevice, s);
  (void)hipMemsetAsync(Dbuf, 0, std::max<size_t>(oD[L], 1) * 8, s);
  (void)hipMemsetAsync(Bbuf, 0, std::max<size_t>(oB[L], 1) * 8, s);
  (void)hipMemsetAsync(bad, 0, sizeof(int), s);
  if (mv.nnzb > 0) {
    const int nb = (mv.nnzb + WG - 1) / WG;
    if (D == 2) k_level_scatter<2><<<nb, WG, 0, s>>>(mv, hb, lev_d, loff_d, oD_d, oB_d, Dbuf, Bbuf);
    else k_level_scatter<3><<<nb, WG, 0, s>>>(mv, hb, lev_d, loff_d, oD_d, oB_d, Dbuf, Bbuf);
  }
  // block LDL^T: S_l in place of D_l (then inverted in place), F_l in place of B_l
  for (int l = 0; l < L; ++l) {
    double* Dl = Dbuf + oD[l];
    if (l > 0) {
      double* Bl = Bbuf + oB[l];
      const double* Sprev = Dbuf + oD[l - 1];
      dgemm(false, false, n[l], n[l - 1], n[l - 1], 1.0, Bl, n[l - 1], Sprev, n[l - 1], 0.0, tmp, n[l - 1], s);
      dgemm(false, true, n[l], n[l], n[l - 1], -1.0, tmp, n[l - 1], Bl, n[l - 1], 1.0, Dl, n[l], s);
      scale_copy(Bl, n[l - 1], tmp, n[l - 1], n[l], n[l - 1], 1.0, s);
    }
    gj_inverse(Dl, n[l], tmp, pivot, bad, s);
  }
  int hbad = 0;
  (void)hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, s);
  (void)hipStreamSynchronize(s);
  if (hbad) {
    release();
    return 1;
  }
  // panels: column block q of Z, then the basis rows of level q
  for (int q = 0; q < L; ++q) {
    const int nq = n[q];
    auto rowsP = [&](int l) { return P + (size_t)loff_h[l] * D * nq; };
    auto rowsQ = [&](int l) { return Q + (size_t)loff_h[l] * D * nq; };
    scale_copy(rowsQ(q), nq, Dbuf + oD[q], nq, nq, nq, 1.0, s);                 // Z_q = S_q^{-1}
    if (q + 1 < L) scale_copy(rowsP(q + 1), nq, Bbuf + oB[q + 1], nq, n[q + 1], nq, -1.0, s);  // Y = -F
    for (int l = q + 2; l < L; ++l)
      dgemm(false, false, n[l], nq, n[l - 1], -1.0, Bbuf + oB[l], n[l - 1], rowsP(l - 1), nq, 0.0, rowsP(l), nq, s);
    for (int l = q + 1; l < L; ++l)
      dgemm(false, false, n[l], nq, n[l], 1.0, Dbuf + oD[l], n[l], rowsP(l), nq, 0.0, rowsQ(l), nq, s);
    for (int l = L - 2; l >= 0; --l)
      dgemm(true, false, n[l], nq, n[l + 1], -1.0, Bbuf + oB[l + 1], n[l], rowsQ(l + 1), nq, l >= q ? 1.0 : 0.0,
            rowsQ(l), nq, s);
    const int sq = n[q] / D;
    if (nf > 1 && sq > 0) {
      const dim3 g((nf + WG - 1) / WG, sq);
      if (D == 2) k_basis_from_panel<2><<<g, WG, 0, s>>>(Q, nq, loff_h[q], nf, mv.bvert, Ud, Uf);
      else k_basis_from_panel<3><<<g, WG, 0, s>>>(Q, nq, loff_h[q], nf, mv.bvert, Ud, Uf);
    }
  }
  const hipError_t e = hipStreamSynchronize(s);
  release();
  return e == hipSuccess ? 0 : 2;
}

}  // namespace cc
