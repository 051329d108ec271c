// FP64 pseudo-inverse solve of the sample-space system (App. F): with
// T = V diag(w) V^T, x = sum over w_i > cutoff * max(w) of v_i (v_i^T b) / w_i.
//
//   1. Householder tridiagonalisation T = Q J Q^T in panels of TNB columns
//      (each column: update from the panel, reflector, b <- H b, and the
//      product of the trailing matrix with the reflector; a rank-2 TNB
//      update of the trailing matrix after each panel).  Reflector j is kept
//      in row j of the working copy, to the right of the diagonal.
//   2. Divide and conquer on J (Cuppen's tearing into halves down to single
//      rows; rank-one merges solved through the secular equation, with the
//      eigenvector formula of Gu and Eisenstat).  The eigenvector matrix is
//      never formed: each merge keeps its permutation, deflation rotations
//      and the K x K matrix U of its non-deflated eigenvectors, and vectors
//      are carried up (c = Z^T Q^T b) and down (y = Z t) the tree.
//   3. t = c / w on the kept eigenvalues, y = Z t, x = Q y.
// Each merge runs on one workgroup per node for the sequential parts (deflation
// scan, rotations), on a thread per entry for the order, and on one wavefront
// per root, entry or column for the secular equations and eigenvectors.
#include "mm.hpp"
#include "model.hpp"
#include <cmath>
#include <vector>

namespace minsr {

// panel width of the tridiagonalisation: the panel vectors that a column
// reads grow with it (k_tri_row 3.9 us at position 0, 4.1 in the second
// half), the number of trailing rank-2 TNB updates (22 us) with its inverse
constexpr int TNB = 16;
constexpr int PINV_MAX_N = 4096;
constexpr int BKB = 64;                    // reflectors of a back-transformation block

// ------------------------------------------------------------ workspace
struct PinvWs {
  // tridiagonalisation
  double *A, *V, *W, *tau, *d, *e, *bq, *y, *s12, *scal, *col, *pd;
  // back-transformation: products of each block's reflectors, their products with x
  double *bg, *sv;
  // divide and conquer, per depth parity (ping-pong)
  double *ev[2], *fr[2], *lr[2], *cv[2], *tv[2];
  // per-merge scratch, indexed by position in [0, n)
  double *es, *dl, *wv, *dlo, *taus, *zh, *uk, *rho, *tk;
  // per-level records (depth l at offset l * n)
  int *perm, *wpos, *rotp, *rotn, *kinfo;   // kinfo: [level][2 * slot]: K, nrot
  double *rotc, *rots;
  double* U;
};

static int depth_of(int n) {
  int D = 0;
  while ((1 << D) < n) ++D;
  return D;
}
static size_t mmax_of(int n, int lev) { return ((size_t)n + ((size_t)1 << lev) - 1) >> lev; }
static size_t u_level_elems(int n, int lev) {
  const size_t mm = mmax_of(n, lev);
  return ((size_t)1 << lev) * mm * mm;
}

size_t pinv_workspace_doubles(int nmax) {
  if (nmax <= 0) return 0;
  const size_t n = (size_t)nmax;
  const int D = depth_of(nmax) + 1;
  size_t u = 0;
  for (int l = 0; l < D; ++l) u += u_level_elems(nmax, l);
  size_t dbl = n * n + (n + BKB - 1) / BKB * BKB * BKB + BKB    // back-transformation
             + 2 * TNB * n + 7 * n + 2 * TNB + 8   // tridiagonalisation
             + 10 * n                                      // ping-pong arrays
             + 11 * n                                      // merge scratch (uk has 3 n)
             + 2 * D * n                                   // rotation coefficients
             + u;
  size_t ints = 4 * (size_t)D * n + 2 * (size_t)D * 2 * n;
  return dbl + (ints + 1) / 2 + 64;
}

static PinvWs carve(double* base, int n, int nmax) {
  PinvWs w;
  const size_t N = (size_t)nmax;
  const int D = depth_of(nmax) + 1;
  double* p = base;
  auto take = [&](size_t k) { double* r = p; p += k; return r; };
  w.A = take(N * N);
  w.V = take(TNB * N); w.W = take(TNB * N);
  w.tau = take(N); w.d = take(N); w.e = take(N); w.bq = take(N); w.y = take(N);
  w.s12 = take(2 * TNB); w.scal = take(8); w.col = take(N); w.pd = take(N);
  w.bg = take((N + BKB - 1) / BKB * BKB * BKB); w.sv = take(BKB);
  for (int i = 0; i < 2; ++i) { w.ev[i] = take(N); w.fr[i] = take(N); w.lr[i] = take(N);
                                w.cv[i] = take(N); w.tv[i] = take(N); }
  w.es = take(N); w.dl = take(N); w.wv = take(N); w.dlo = take(N); w.taus = take(N);
  w.zh = take(N); w.uk = take(3 * N); w.rho = take(N); w.tk = take(N);
  w.rotc = take((size_t)D * N); w.rots = take((size_t)D * N);
  size_t u = 0;
  for (int l = 0; l < D; ++l) u += u_level_elems(nmax, l);
  w.U = take(u);
  int* q = reinterpret_cast<int*>(p);
  w.perm = q; q += (size_t)D * N;
  w.wpos = q; q += (size_t)D * N;
  w.rotp = q; q += (size_t)D * N;
  w.rotn = q; q += (size_t)D * N;
  w.kinfo = q;
  (void)n;
  return w;
}

// ------------------------------------------------------------ helpers
// (an xor butterfly's sums without its round trips through the shared-memory
// crossbar: every kernel here waits for one to three of them in a row)
__device__ __forceinline__ double wave_sum(double v) { return unit_sum<64>(v); }
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = fmax(v, __shfl_xor(v, m, 64));
  return v;
}
// sum over a workgroup of up to 1024 threads; every thread gets the result
__device__ double block_sum(double v, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < nw; ++i) s += red[i];
  return s;
}
__device__ double block_max(double v, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  v = wave_max(v);
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double s = red[0];
  for (int i = 1; i < nw; ++i) s = fmax(s, red[i]);
  return s;
}

// node `slot` of depth `lev`: halving from the root [0, n)
__device__ __host__ inline void node_of(int n, int lev, int slot, int& lo, int& m) {
  lo = 0; m = n;
  for (int b = lev - 1; b >= 0; --b) {
    const int half = m / 2;
    if ((slot >> b) & 1) { lo += half; m -= half; }
    else m = half;
  }
}

// ================================================== tridiagonalisation
// Two launches a column.  Every launch waits for the one before it, so a
// column's time is two launches, their loads' latencies and the stream of the
// trailing matrix through k_tri_mv; both kernels therefore run on as many
// workgroups as there are rows for, form the scalars redundantly from
// partial sums, and request every operand before the first wait.  (With the
// reflector, the panel's dot products and w on one workgroup the two kernels
// took 9.7 + 10.8 us on average at n = 4096; now 3.8 + 10.3,
// and 22 instead of 2 x 19 us for the update of 16 columns.)
struct TriArgs {
  double *A, *V, *W, *tau, *d, *e, *bq, *y, *s12, *col, *pd, *pn, *pb, *scal;
  int n;
};

constexpr int TBS = 1024;
constexpr int TMR = 4;                     // rows (wavefronts) of a k_tri_mv workgroup: 4 10.6 us
                                           // a column of n = 4096, 8 11.0, 16 12.7

// value of lane q (a constant) in every lane
__device__ __forceinline__ double lane_value(double v, int q) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, q);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), q);
  return __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}

// Rows i > j, one per thread, after column j's product y = A v (panel position
// p): g = y - sum_{q<p} V_q s1[q] + W_q s2[q], w = tau g + alpha v with alpha =
// -tau^2 / 2 g.v and g.v = y.v - 2 s1.s2; the right-hand side's reflection;
// then column j + 1 of the updated matrix, A[j+1][i] - sum_{q<=p} V_q[i]
// W_q[j+1] + W_q[i] V_q[j+1], and this workgroup's parts of its norm and of its
// product with the right-hand side, rows j + 3 onwards.  p < 0: column 0 as it
// is.  Q is p rounded up.
template <int Q>
__global__ __launch_bounds__(64) void k_tri_row(TriArgs a, int j, int p, int npd) {
  const int n = a.n, lane = threadIdx.x;
  const int i = j + 1 + 64 * blockIdx.x + lane, ii = min(i, n - 1);
  double vq[Q ? Q : 1], wq[Q ? Q : 1];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const size_t o = (size_t)(q < p ? q : 0) * n + ii;
    vq[q] = a.V[o];
    wq[q] = a.W[o];
  }
  const double aj = a.A[(size_t)(j + 1) * n + ii], b0 = a.bq[ii];
  double w = 0.0, vi = 0.0, Wj = 0.0, vb = 0.0, col = aj;
  if (p >= 0) {
    const int lq = lane < p ? lane : 0;
    double l1 = a.s12[lq], l2 = a.s12[TNB + lq];
    double lv = a.V[(size_t)lq * n + j + 1], lw = a.W[(size_t)lq * n + j + 1];
    const double yi = a.y[ii], yj = a.y[j + 1], tp = a.tau[j];
    vi = a.V[(size_t)p * n + ii];
    vb = a.scal[1];
    double sp = 0.0;
#pragma unroll
    for (int k = 0; k < PINV_MAX_N / TMR / 64; ++k) {
      const double x = a.pd[min(lane + 64 * k, npd - 1)];
      sp += lane + 64 * k < npd ? x : 0.0;
    }
    if (lane >= p) l1 = l2 = lv = lw = 0.0;
    const double alpha = -0.5 * tp * tp * wave_sum(sp - 2.0 * (l1 * l2));
    Wj = tp * (yj - wave_sum(lv * l1 + lw * l2)) + alpha;       // v[j+1] = 1
    double g = 0.0, c = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const double v_ = q < p ? vq[q] : 0.0, w_ = q < p ? wq[q] : 0.0;
      g = fma(w_, lane_value(l2, q), fma(v_, lane_value(l1, q), g));
      c = fma(w_, lane_value(lv, q), fma(v_, lane_value(lw, q), c));
    }
    w = tp * (yi - g) + alpha * vi;
    col = (aj - c) - (vi * Wj + w);
  }
  const double b = b0 - vb * vi;
  if (i < n) {
    if (p >= 0) a.W[(size_t)p * n + i] = w;
    a.col[i] = col;
    a.bq[i] = b;
    if (i == j + 1) a.d[i] = col;
  }
  const double x = i >= j + 3 && i < n ? col : 0.0;
  const double pn = wave_sum(x * x), pb = wave_sum(x * b);
  if (lane == 0) { a.pn[blockIdx.x] = pn; a.pb[blockIdx.x] = pb; }
}

// The reflector of column j (position p of its panel) from col, formed by
// every workgroup: v = col sc with v[j+1] = 1, in LDS.  Then one wavefront a
// row: y[i] = A[i] . v for i > j; and, as 2p more rows, s1[q] = W_q . v and
// s2[q] = V_q . v.  nrow workgroups take A's rows, workgroup b rows 4 (rb + b)
// onwards with rb a multiple of 8: a row stays on the same XCD from column to
// column, so that trailing matrices within the L2 caches stay there.
__global__ __launch_bounds__(64 * TMR) void k_tri_mv(TriArgs a, int j, int p, int rb, int nrow,
                                                     int npn) {
  __shared__ double vs[PINV_MAX_N];
  __shared__ double pdw[TMR];
  const int n = a.n, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int len = n - j - 1, blk = blockIdx.x;
  const bool tail = blk >= nrow;
  const int i = TMR * (rb + blk) + wv;                     // row of A
  const int q = TMR * (blk - nrow) + wv;                   // or panel vector
  const bool on = tail ? q < 2 * p : i > j && i < n;
  if (!tail && TMR * (rb + blk) + TMR - 1 <= j) return;    // no rows: the whole workgroup
  const double* row = (!on ? a.A + (size_t)(j + 1) * n
                       : !tail ? a.A + (size_t)i * n
                       : q < p ? a.W + (size_t)q * n : a.V + (size_t)(q - p) * n) + j + 1;
  // the first 1024 columns, and column j with its partial sums
  double r[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) r[t] = row[min(lane + 64 * t, len - 1)];
  const double x0 = a.col[j + 1], b0 = a.bq[j + 1];
  const double pn = a.pn[min(lane, npn - 1)], pb = a.pb[min(lane, npn - 1)];
  constexpr int PT = PINV_MAX_N / (64 * TMR);
  double cl[PT];
#pragma unroll
  for (int u = 0; u < PT; ++u) cl[u] = a.col[j + 1 + min(tid + 64 * TMR * u, len - 1)];
  const double sig2 = wave_sum(lane < npn ? pn : 0.0), cb = wave_sum(lane < npn ? pb : 0.0);
  double t, beta, sc;
  if (sig2 == 0.0) { t = 0.0; beta = x0; sc = 0.0; }
  else {
    beta = -copysign(sqrt(x0 * x0 + sig2), x0);
    t = (beta - x0) / beta;
    sc = 1.0 / (x0 - beta);
  }
#pragma unroll
  for (int u = 0; u < PT; ++u) {
    const int k = tid + 64 * TMR * u;
    vs[k] = k == 0 ? 1.0 : k < len ? cl[u] * sc : 0.0;
  }
  __syncthreads();
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  for (int c = 0; c < len; c += 1024) {
    double x[16];
    if (c + 1024 < len) {
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = row[min(c + 1024 + lane + 64 * u, len - 1)];
    }
#pragma unroll
    for (int u = 0; u < 16; u += 4) {
      const double* v = vs + c + lane + 64 * u;
      s0 = fma(r[u], v[0], s0);
      s1 = fma(r[u + 1], v[64], s1);
      s2 = fma(r[u + 2], v[128], s2);
      s3 = fma(r[u + 3], v[192], s3);
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) r[u] = x[u];
  }
  const double y = wave_sum((s0 + s1) + (s2 + s3));
  if (tail) {
    if (on && lane == 0) a.s12[q < p ? q : TNB + q - p] = y;
    return;
  }
  if (lane == 0) {
    const double vi = on ? vs[i - j - 1] : 0.0;
    if (on) {
      a.y[i] = y;
      a.V[(size_t)p * n + i] = vi;
      a.A[(size_t)j * n + i] = vi;
    }
    pdw[wv] = vi * y;
  }
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < TMR; ++w) s += pdw[w];
    a.pd[rb + blk - (j + 1) / TMR] = s;
    if (TMR * (rb + blk) <= j + 1) {       // the workgroup of row j + 1
      a.tau[j] = t;
      a.e[j] = beta;
      a.scal[1] = t * (b0 + sc * cb);
    }
  }
}

// A[i][c] -= sum_q V[q][i] W[q][c] + W[q][i] V[q][c], i, c >= j1: 64 x 64
// tiles on the FP64 matrix cores.  Wave w takes rows 16 w .. 16 w + 15 of
// the tile as four 16 x 16 blocks; the product's K index runs over the 2 TNB
// panel columns [V W] against [W V] (zero beyond nb and beyond n).  Lane l
// of v_mfma_f64_16x16x4 supplies A[l % 16][l / 16] and B[l / 16][l % 16]
// and holds D[l / 16 + 4 e][l % 16] in element e.
typedef double f64x4_e __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_tri_syr2k(double* A, const double* V, const double* W,
                                                   int n, int j1, int nb) {
  __shared__ double Vi[TNB][64], Wi[TNB][64], Vc[TNB][64], Wc[TNB][64];
  const int r0 = j1 + blockIdx.y * 64, c0 = j1 + blockIdx.x * 64, tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  for (int e = tid; e < TNB * 64; e += 256) {
    const int q = e / 64, k = e % 64;
    const bool okq = q < nb;
    Vi[q][k] = (okq && r0 + k < n) ? V[(size_t)q * n + r0 + k] : 0.0;
    Wi[q][k] = (okq && r0 + k < n) ? W[(size_t)q * n + r0 + k] : 0.0;
    Vc[q][k] = (okq && c0 + k < n) ? V[(size_t)q * n + c0 + k] : 0.0;
    Wc[q][k] = (okq && c0 + k < n) ? W[(size_t)q * n + c0 + k] : 0.0;
  }
  // this lane's 16 elements of the tile, requested before the barrier
  f64x4_e acc[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = r0 + 16 * w + (lane >> 4) + 4 * e, c = c0 + 16 * cb + (lane & 15);
      acc[cb][e] = (r < n && c < n) ? A[(size_t)r * n + c] : 0.0;
    }
  __syncthreads();
  const int i = 16 * w + (lane & 15);
#pragma unroll
  for (int ks = 0; ks < 2 * TNB; ks += 4) {
    const int k = ks + (lane >> 4);
    const double a = k < TNB ? Vi[k][i] : Wi[k - TNB][i];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const int c = 16 * cb + (lane & 15);
      const double b = k < TNB ? Wc[k][c] : Vc[k - TNB][c];
      acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a, b, acc[cb], 0, 0, 0);
    }
  }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = r0 + 16 * w + (lane >> 4) + 4 * e, c = c0 + 16 * cb + (lane & 15);
      if (r < n && c < n) A[(size_t)r * n + c] = acc[cb][e];
    }
}

__global__ void k_pinv_copy(const double* T, double* A, size_t nn, const double* b, double* bq,
                            int n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nn) A[i] = T[i];
  if (i < (size_t)n) bq[i] = b[i];
}

// x = H_0 H_1 ... H_{n-2} y, last reflector first, in blocks of BKB: with the
// block's reflectors as rows of V, H_j0 ... H_j0+63 = I - V^T Z V where z = Z s
// solves z_j = tau_j (s_j - sum_{k>j} (v_j . v_k) z_k), s = V x.  The products
// v_j . v_k of all blocks are formed beforehand (k_back_gram); then a block
// takes two launches.  (One reflector after the other, on one workgroup: 8.4
// ms at n = 4096; this: 0.86
// ms.)

// entry i of reflector j (row j of A, right of the diagonal)
__device__ __forceinline__ double refl(const double* A, int n, int j, int i) {
  const bool ok = i > j && i < n && j < n - 1;
  const double v = A[ok ? (size_t)j * n + i : 0];
  return ok ? v : 0.0;
}

// products of block b's reflectors: 16 of them against the block, the columns
// split over the four wavefronts.  A lane's four columns of a 16-column step
// are consecutive, so a row's step is one 128-byte line.
__global__ __launch_bounds__(256) void k_back_gram(const double* A, double* G, int n) {
  __shared__ double part[4][16][BKB];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, m = lane & 15, g = lane >> 4;
  const int j0 = blockIdx.x * BKB, ja = j0 + 16 * blockIdx.y;
  f64x4_e acc[4] = {};
  for (int k0 = j0 + 16 * w; k0 < n; k0 += 64) {
    double x[4], y[4][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = refl(A, n, ja + m, k0 + 4 * g + e);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) y[t][e] = refl(A, n, j0 + 16 * t + m, k0 + 4 * g + e);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[e], y[t][e], acc[t], 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) part[w][g + 4 * e][16 * t + m] = acc[t][e];
  __syncthreads();
  for (int q = threadIdx.x; q < 16 * BKB; q += 256) {
    const int r = q / BKB, c = q % BKB;
    G[((size_t)blockIdx.x * BKB + 16 * blockIdx.y + r) * BKB + c] =
        (part[0][r][c] + part[1][r][c]) + (part[2][r][c] + part[3][r][c]);
  }
}

// s_j = v_j . x, one workgroup per reflector of the block
__global__ __launch_bounds__(256) void k_back_dot(const double* A, const double* x, double* sv,
                                                  int n, int j0) {
  __shared__ double red[4];
  const int j = j0 + blockIdx.x;
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < PINV_MAX_N / 256; ++u) {
    const int i = j0 + 1 + threadIdx.x + 256 * u;
    s = fma(refl(A, n, j, i), x[min(i, n - 1)], s);
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) sv[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// x = x - V^T z, 64 entries a workgroup; every workgroup solves for z
__global__ __launch_bounds__(64) void k_back_upd(const double* A, const double* tau,
                                                 const double* G, const double* sv,
                                                 const double* xin, double* x, int n, int j0) {
  const int lane = threadIdx.x, i = blockIdx.x * 64 + lane;
  double gk[BKB], v[BKB];
#pragma unroll
  for (int k = 0; k < BKB; ++k) gk[k] = G[(size_t)(j0 + k) * BKB + lane];
#pragma unroll
  for (int k = 0; k < BKB; ++k) v[k] = refl(A, n, j0 + k, i);
  const double t = j0 + lane < n - 1 ? tau[j0 + lane] : 0.0;
  double s = sv[lane], xi = xin[min(i, n - 1)];
#pragma unroll
  for (int k = BKB - 1; k >= 0; --k) {
    const double z = lane_value(t * s, k);
    s = fma(-gk[k], z, s);             // lanes above k are done
    xi = fma(-v[k], z, xi);
  }
  if (i < n) x[i] = xi;
}

// ================================================== divide and conquer
struct DcArgs {
  PinvWs w;
  int n, nmax, D;
  size_t ubase;     // U offset of the level
  size_t umm;       // slot stride of U at the level (mmax^2)
  double cutoff;
  uint32_t* status;
};

// scale J to unit max norm; leaves of depth D: torn diagonal, first/last
// rows 1, right-hand side b' = Q^T b
__global__ __launch_bounds__(TBS) void k_dc_init(DcArgs a) {
  __shared__ double red[TBS / 64];
  const int n = a.n, tid = threadIdx.x;
  double mx = 0.0;
  for (int i = tid; i < n; i += TBS) {
    mx = fmax(mx, fabs(a.w.d[i]));
    if (i < n - 1) mx = fmax(mx, fabs(a.w.e[i]));
  }
  mx = block_max(mx, red);
  // a non-finite entry (NaN compares false) makes the result meaningless:
  // flag it; the later kernels stay in bounds either way
  bool bad = !(mx <= 1.7976931348623157e308);
  if (bad && tid == 0 && a.status) atomicOr(a.status, MINSR_ST_EIG_NOCONV);
  const double scale = (mx > 0.0 && !bad) ? mx : 1.0;
  const double inv = 1.0 / scale;
  const int P = a.D & 1;
  for (int i = tid; i < n; i += TBS) {
    const double ei = i < n - 1 ? a.w.e[i] * inv : 0.0;
    const double em = i > 0 ? a.w.e[i - 1] * inv : 0.0;
    a.w.es[i] = ei;
    a.w.ev[P][i] = a.w.d[i] * inv - fabs(em) - fabs(ei);
    a.w.fr[P][i] = 1.0;
    a.w.lr[P][i] = 1.0;
    a.w.cv[P][i] = a.w.bq[i];
  }
  if (tid == 0) a.w.scal[0] = scale;
}

constexpr int DCB = 1024;   // workgroup of the per-node kernels

// sum of v over the lower threads of a DCB workgroup, and over all of it
__device__ int block_before(int v, int* wsum, int& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const int y = __shfl_up(x, m, 64);
    if (lane >= m) x += y;
  }
  __syncthreads();
  if (lane == 63) wsum[wv] = x;
  __syncthreads();
  int before = 0, all = 0;
  for (int i = 0; i < DCB / 64; ++i) {
    before += i < wv ? wsum[i] : 0;
    all += wsum[i];
  }
  total = all;
  return before + x - v;
}

// Ascending order of every node's children's eigenvalues (ties by index), one
// entry per thread: m compares each, on as many compute units as there are 64
// entries (inside k_dc_prep, on one: 1.1 of its 1.55 ms at 4096 entries).
__global__ __launch_bounds__(64) void k_dc_rank(DcArgs a, int lev) {
  extern __shared__ double ranked[];
  const int tid = threadIdx.x, slot = blockIdx.y;
  int lo, m;
  node_of(a.n, lev, slot, lo, m);
  const int i = blockIdx.x * 64 + tid;
  if (m < 2 || (int)blockIdx.x * 64 >= m) return;
  const double* ev = a.w.ev[(lev + 1) & 1] + lo;
  for (int k = tid; k < m; k += 64) {
    const double v = ev[k];
    ranked[k] = v == v ? v : INFINITY;   // NaN ranks as +inf, so ranks stay a permutation
  }
  __syncthreads();
  if (i >= m) return;
  const double di = ranked[i];
  int r = 0;
#pragma unroll 8
  for (int k = 0; k < m; ++k) {
    const double dk = ranked[k];
    r += (dk < di) || (dk == di && k < i);
  }
  a.w.perm[(size_t)lev * a.nmax + lo + r] = i;
}

// One workgroup per node of depth lev: gather the children's eigenvalues and
// rank-one vector in their order, deflate (small z, then close pairs by a rotation),
// record the permutation, positions and rotations, and carry the first/last
// rows and c into the node's basis up to the K x K block.
__global__ __launch_bounds__(DCB) void k_dc_prep(DcArgs a, int lev) {
  extern __shared__ double sm[];
  __shared__ double red[DCB / 64];
  __shared__ uint64_t flags[PINV_MAX_N / 64];
  __shared__ int wsum[DCB / 64];
  __shared__ int sK, sR;
  const int n = a.n, tid = threadIdx.x, slot = blockIdx.x;
  int lo, m;
  node_of(n, lev, slot, lo, m);
  if (m == 0) return;
  const int Pc = (lev + 1) & 1, P = lev & 1;
  const PinvWs& w = a.w;
  int* kinfo = w.kinfo + (size_t)lev * 4 * a.nmax;
  if (m == 1) {
    if (tid == 0) {
      w.ev[P][lo] = w.ev[Pc][lo];
      w.fr[P][lo] = 1.0;
      w.lr[P][lo] = 1.0;
      w.cv[P][lo] = w.cv[Pc][lo];
      kinfo[2 * slot] = -1;
      kinfo[2 * slot + 1] = 0;
    }
    return;
  }
  double* sd = sm;            // [m] d, sorted
  double* sz = sm + m;        // [m] z, sorted
  double* s3 = sm + 2 * m;    // [m] scratch
  const int m1 = m / 2;
  const double beta = w.es[lo + m1 - 1];
  const double rho = 2.0 * fabs(beta);
  const double sg = beta >= 0.0 ? 1.0 : -1.0;
  const int* perm = w.perm + (size_t)lev * a.nmax + lo;
  int* wpos = w.wpos + (size_t)lev * a.nmax + lo;
  int* rotp = w.rotp + (size_t)lev * a.nmax + lo;
  int* rotn = w.rotn + (size_t)lev * a.nmax + lo;
  double* rotc = w.rotc + (size_t)lev * a.nmax + lo;
  double* rots = w.rots + (size_t)lev * a.nmax + lo;
  double mx = 0.0;
  for (int r = tid; r < m; r += DCB) {
    const int i = perm[r];
    const double v = w.ev[Pc][lo + i];
    sd[r] = v == v ? v : INFINITY;
    const double zi = (i < m1 ? w.lr[Pc][lo + i] : sg * w.fr[Pc][lo + i]) * 0.70710678118654752440;
    sz[r] = zi;
    mx = fmax(mx, fmax(fabs(sd[r]), fabs(zi)));
  }
  mx = block_max(mx, red);
  const double tol = 8.0 * 2.220446049250313e-16 * mx;
  // Deflation, as a scan over the entries in order: entries of small z are
  // dropped, and of two neighbours left that are close the first one is rotated
  // away.  Whether unrotated neighbours are close is decided in parallel; one
  // thread follows only the chains of rotations (in a scan by one thread every
  // entry waited for its root and divisions: 4096 entries of a random matrix
  // 880 us, now 29; a step's spectrum has more rotations: 10 x 10, 4096 samples
  // 0.80 ms over the twelve levels).
  auto close = [&](int pa, int pb, double& tt, double& c_, double& s_) {
    s_ = sz[pa];
    c_ = sz[pb];
    tt = hypot(c_, s_);
    const double t = sd[pb] - sd[pa];
    c_ /= tt; s_ = -s_ / tt;
    return fabs(t * c_ * s_) <= tol;
  };
  int* left = reinterpret_cast<int*>(s3);      // [m] entries left, in order
  int* gone = left + m;                        // [m] rotated away
  const int ch = (m + DCB - 1) / DCB, i0 = min(tid * ch, m), i1 = min(i0 + ch, m);
  int cnt = 0, S;
  for (int i = i0; i < i1; ++i) cnt += !(rho * fabs(sz[i]) <= tol);
  const int first = block_before(cnt, wsum, S);
  for (int i = i0, at = first; i < i1; ++i)
    if (!(rho * fabs(sz[i]) <= tol)) { left[at] = i; gone[at] = 0; ++at; }
  __syncthreads();
  for (int q0 = 0; q0 < S; q0 += DCB) {
    const int q = q0 + tid;
    double tt, c_, s_;
    const uint64_t bits = __ballot(q + 1 < S && close(left[min(q, S - 1)], left[min(q + 1, S - 1)], tt, c_, s_));
    if ((tid & 63) == 0) flags[q >> 6] = bits;
  }
  __syncthreads();
  if (tid == 0) {
    int nr = 0, cur = 0;
    for (int wd = 0; 64 * wd < S; ++wd)
      for (uint64_t bits = flags[wd]; bits; bits &= bits - 1) {
        int e = 64 * wd + __builtin_ctzll(bits);
        if (e < cur) continue;
        for (; e + 1 < S; ++e) {
          const int pa = left[e], pb = left[e + 1];
          double tt, c_, s_;
          if (!close(pa, pb, tt, c_, s_)) break;
          sz[pb] = tt; sz[pa] = 0.0;
          rotp[nr] = pa; rotn[nr] = pb; rotc[nr] = c_; rots[nr] = s_; ++nr;
          const double dp = sd[pa], dn = sd[pb];
          sd[pa] = dp * c_ * c_ + dn * s_ * s_;
          sd[pb] = dp * s_ * s_ + dn * c_ * c_;
          gone[e] = 1;
        }
        cur = e + 1;
      }
    sK = S - nr; sR = nr;
    kinfo[2 * slot] = S - nr;
    kinfo[2 * slot + 1] = nr;
    w.rho[lo] = rho;
  }
  __syncthreads();
  // wpos = [not deflated ..., small z ..., rotated away ...]
  {
    const int e0 = min(tid * ch, S), e1 = min(e0 + ch, S);
    int kept = 0, all;
    for (int e = e0; e < e1; ++e) kept += !gone[e];
    int at = block_before(kept, wsum, all);
    for (int e = e0; e < e1; ++e) {
      if (gone[e]) wpos[sK + (m - S) + (e - at)] = left[e];
      else wpos[at++] = left[e];
    }
    for (int i = i0, ls = first; i < i1; ++i) {
      if (ls < S && left[ls] == i) ++ls;
      else wpos[sK + (i - ls)] = i;
    }
  }
  __syncthreads();
  const int K = sK, nr = sR;
  for (int k = tid; k < m; k += DCB) {
    const int p = wpos[k];
    if (k < K) { w.dl[lo + k] = sd[p]; w.wv[lo + k] = sz[p]; }
    else w.ev[P][lo + k] = sd[p];
  }
  // carry fr = [fr_left; 0], lr = [0; lr_right], c into working order,
  // rotate, reorder to k order; deflated parts are the node's outputs
  __syncthreads();
  for (int vsel = 0; vsel < 3; ++vsel) {
    for (int r = tid; r < m; r += DCB) {
      const int i = perm[r];
      double val;
      if (vsel == 0) val = i < m1 ? w.fr[Pc][lo + i] : 0.0;
      else if (vsel == 1) val = i >= m1 ? w.lr[Pc][lo + i] : 0.0;
      else val = w.cv[Pc][lo + i];
      s3[r] = val;
    }
    __syncthreads();
    if (tid == 0) {
      for (int t = 0; t < nr; ++t) {
        const int pa = rotp[t], pb = rotn[t];
        const double c_ = rotc[t], s_ = rots[t];
        const double wa = s3[pa], wb = s3[pb];
        s3[pa] = c_ * wa + s_ * wb;
        s3[pb] = -s_ * wa + c_ * wb;
      }
    }
    __syncthreads();
    double* outv = vsel == 0 ? w.fr[P] : (vsel == 1 ? w.lr[P] : w.cv[P]);
    for (int k = tid; k < m; k += DCB) {
      const double val = s3[wpos[k]];
      if (k < K) w.uk[(size_t)vsel * a.nmax + lo + k] = val;
      else outv[lo + k] = val;
    }
    __syncthreads();
  }
}

// Secular equation 1 + rho sum_i w_i^2 / (dl_i - lambda) = 0 for root j of
// every node at depth lev, in tau = lambda - dl_origin, to neighbouring values
// of tau between which its computed sign changes.  One wavefront per root; the
// node's poles and weights are staged in LDS.  A few steps that keep the pole
// at the origin and take the rest of the sum as linear (a quadratic each,
// inside the bracket or else its middle) bring the bracket to a few units in
// the last place, bisection does the rest: about a dozen sums instead of sixty
// (n = 4096, sum over the levels 1.9 -> 1.3 ms; n = 1000 0.15 ms of 9).
constexpr int SEC_WAVES = 16;
__global__ __launch_bounds__(64 * SEC_WAVES) void k_dc_secular(DcArgs a, int lev) {
  extern __shared__ double sm[];
  const int slot = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  int lo, m;
  node_of(a.n, lev, slot, lo, m);
  const int* kinfo = a.w.kinfo + (size_t)lev * 4 * a.nmax;
  if (m < 2) return;
  const int K = kinfo[2 * slot];
  const int j0 = blockIdx.x * SEC_WAVES;
  if (K <= 0 || j0 >= K) return;
  double* pd = sm;
  double* pw = sm + K;
  for (int i = tid; i < K; i += 64 * SEC_WAVES) {
    pd[i] = a.w.dl[lo + i];
    const double wi = a.w.wv[lo + i];
    pw[i] = wi * wi;
  }
  __syncthreads();
  const int j = j0 + (tid >> 6);
  if (j >= K) return;
  const double rho = a.w.rho[lo];
  int o;
  double tl, th;
  if (j < K - 1) {
    const double mid = 0.5 * (pd[j] + pd[j + 1]);
    double s = 0.0;
    for (int i = lane; i < K; i += 64) s += pw[i] / (pd[i] - mid);
    s = wave_sum(s);
    if (1.0 + rho * s > 0.0) { o = j; tl = 0.0; th = mid - pd[j]; }
    else { o = j + 1; tl = mid - pd[j + 1]; th = 0.0; }
  } else {
    double s = 0.0;
    for (int i = lane; i < K; i += 64) s += pw[i];
    s = wave_sum(s);
    o = j; tl = 0.0; th = rho * s;
  }
  const double dorg = pd[o];
  const double wo = rho * pw[o], eps = 2.220446049250313e-16;
  double t = 0.5 * (tl + th);
  double step = INFINITY;                          // the last one
  for (int it = 0; it < 10 && step > 8.0 * eps * fabs(t); ++it) {
    double s = 0.0, r = 0.0, r1 = 0.0;             // the sum; without the origin; its slope
    for (int i = lane; i < K; i += 64) {
      const double d = (pd[i] - dorg) - t, q = pw[i] / d;
      s += q;
      r += i == o ? 0.0 : q;
      r1 += i == o ? 0.0 : q * __builtin_amdgcn_rcp(d);
    }
    s = wave_sum(s); r = wave_sum(r); r1 = rho * wave_sum(r1);
    if (1.0 + rho * s < 0.0) tl = t; else th = t;
    // r1 x^2 + (r - r1 t) x - wo = 0, x on the origin's side
    const double b = 1.0 + rho * r - r1 * t, c = sqrt(b * b + 4.0 * r1 * wo);
    double x = o == j ? 2.0 * wo / (b + c) : -2.0 * wo / (c - b);
    if (!(x > tl && x <= th)) x = 0.5 * (tl + th);
    step = fabs(x - t);
    t = x;
  }
  // the signs on both sides of t, further out if they are equal
  double h = 8.0 * eps * fabs(t) + 2.0 * step;
  for (int it = 0; it < 3; ++it, h *= 64.0) {
    bool above = false, below = false;
    for (int side = 0; side < 2; ++side) {
      const double tm = side == 0 ? t - h : t + h;
      if (!(tm > tl && tm < th)) { (side == 0 ? below : above) = true; continue; }
      double s = 0.0;
      for (int i = lane; i < K; i += 64) s += pw[i] / ((pd[i] - dorg) - tm);
      s = wave_sum(s);
      if (1.0 + rho * s < 0.0) { tl = tm; below = below || side == 0; }
      else { th = tm; above = above || side == 1; }
    }
    if (above && below) break;
  }
  for (int it = 0; it < 400; ++it) {
    const double tm = 0.5 * (tl + th);
    if (tm == tl || tm == th) break;
    double s = 0.0;
    for (int i = lane; i < K; i += 64) s += pw[i] / ((pd[i] - dorg) - tm);
    s = wave_sum(s);
    if (1.0 + rho * s < 0.0) tl = tm; else th = tm;
  }
  if (lane == 0) {
    const double tau = 0.5 * (tl + th);
    a.w.dlo[lo + j] = dorg;
    a.w.taus[lo + j] = tau;
    a.w.ev[lev & 1][lo + j] = dorg + tau;
  }
}

// Gu-Eisenstat: |zhat_i|^2 = (lambda_{K-1} - d_i)/rho
//   * prod_{j<i} (lambda_j - d_i)/(d_j - d_i) * prod_{i<=j<K-1} (lambda_j - d_i)/(d_{j+1} - d_i)
// A wavefront per entry: the product's K divisions are a serial chain for one
// thread (64 us a level of n = 4096, now 6).
__global__ __launch_bounds__(256) void k_dc_zhat(DcArgs a, int lev) {
  const int slot = blockIdx.y, lane = threadIdx.x & 63;
  int lo, m;
  node_of(a.n, lev, slot, lo, m);
  if (m < 2) return;
  const int K = a.w.kinfo[(size_t)lev * 4 * a.nmax + 2 * slot];
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= K) return;
  const double* dl = a.w.dl + lo;
  const double* dlo = a.w.dlo + lo;
  const double* ta = a.w.taus + lo;
  const double di = dl[i];
  double prod = 1.0;
  for (int j = lane; j < K - 1; j += 64) {
    const double num = (dlo[j] - di) + ta[j];
    const double den = (j < i ? dl[j] : dl[j + 1]) - di;
    prod *= num / den;
  }
#pragma unroll
  for (int q = 32; q >= 1; q >>= 1) prod *= __shfl_xor(prod, q, 64);
  prod *= ((dlo[K - 1] - di) + ta[K - 1]) / a.w.rho[lo];
  if (lane == 0) a.w.zh[lo + i] = copysign(sqrt(fmax(prod, 0.0)), a.w.wv[lo + i]);
}

// eigenvector columns of the non-deflated block: u_k = zhat_k / (d_k - lambda_col),
// normalised, stored column-major (K x K) in the node's U slot; the node's
// first/last rows and c follow as dot products with the carried vectors.
__global__ __launch_bounds__(256) void k_dc_ucols(DcArgs a, int lev) {
  const int slot = blockIdx.y, lane = threadIdx.x & 63;
  int lo, m;
  node_of(a.n, lev, slot, lo, m);
  if (m < 2) return;
  const int K = a.w.kinfo[(size_t)lev * 4 * a.nmax + 2 * slot];
  const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= K) return;
  const double* dl = a.w.dl + lo;
  const double* zh = a.w.zh + lo;
  const double dorg = a.w.dlo[lo + col], tau = a.w.taus[lo + col];
  double nn = 0.0;
  for (int k = lane; k < K; k += 64) {
    const double u = zh[k] / ((dl[k] - dorg) - tau);
    nn += u * u;
  }
  const double rn = 1.0 / sqrt(wave_sum(nn));
  double* U = a.w.U + a.ubase + (size_t)slot * a.umm + (size_t)col * K;
  const size_t N = a.nmax;
  double f = 0.0, l = 0.0, c = 0.0;
  for (int k = lane; k < K; k += 64) {
    const double u = zh[k] / ((dl[k] - dorg) - tau) * rn;
    U[k] = u;
    f += u * a.w.uk[lo + k];
    l += u * a.w.uk[N + lo + k];
    c += u * a.w.uk[2 * N + lo + k];
  }
  f = wave_sum(f); l = wave_sum(l); c = wave_sum(c);
  if (lane == 0) {
    const int P = lev & 1;
    a.w.fr[P][lo + col] = f;
    a.w.lr[P][lo + col] = l;
    a.w.cv[P][lo + col] = c;
  }
}

// root: t = c / lambda on the kept eigenvalues (lambda > cutoff * lambda_max)
__global__ __launch_bounds__(TBS) void k_dc_root(DcArgs a) {
  __shared__ double red[TBS / 64];
  const int n = a.n, tid = threadIdx.x;
  double mx = -INFINITY;
  for (int i = tid; i < n; i += TBS) mx = fmax(mx, a.w.ev[0][i]);
  mx = block_max(mx, red);
  const double scale = a.w.scal[0];
  const double thr = a.cutoff * mx;
  for (int i = tid; i < n; i += TBS) {
    const double lam = a.w.ev[0][i];
    a.w.tv[0][i] = (lam > thr && lam > 0.0) ? a.w.cv[0][i] / (lam * scale) : 0.0;
  }
}

// down the tree, node at depth lev: tk = U t (k < K), then working order,
// rotations in reverse, scatter to the children's positions.  64 entries a
// workgroup, the columns dealt to its four wavefronts, eight loads in flight
// (one thread an entry, one load after the other: 106 us a level, now 10).
__global__ __launch_bounds__(256) void k_dc_down_gemv(DcArgs a, int lev) {
  __shared__ double part[4][64];
  const int slot = blockIdx.y, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int lo, m;
  node_of(a.n, lev, slot, lo, m);
  if (m < 2 || (int)blockIdx.x * 64 >= m) return;
  const int K = a.w.kinfo[(size_t)lev * 4 * a.nmax + 2 * slot];
  const int k = blockIdx.x * 64 + lane;
  const double* t = a.w.tv[lev & 1] + lo;
  double s = 0.0;
  if (k < K) {
    const double* U = a.w.U + a.ubase + (size_t)slot * a.umm + k;
    for (int c0 = wv; c0 < K; c0 += 32) {
      double u[8], x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int c = min(c0 + 4 * q, K - 1);
        u[q] = U[(size_t)c * K];
        x[q] = t[c];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) s = c0 + 4 * q < K ? fma(u[q], x[q], s) : s;
    }
  }
  part[wv][lane] = s;
  __syncthreads();
  if (wv == 0 && k < m)
    a.w.tk[lo + k] = k < K ? (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]) : t[k];
}

__global__ __launch_bounds__(DCB) void k_dc_down_post(DcArgs a, int lev) {
  extern __shared__ double sm[];
  const int slot = blockIdx.x, tid = threadIdx.x;
  int lo, m;
  node_of(a.n, lev, slot, lo, m);
  if (m == 0) return;
  const int Pn = (lev + 1) & 1;
  if (m == 1) {
    if (tid == 0) a.w.tv[Pn][lo] = a.w.tv[lev & 1][lo];
    return;
  }
  const int* kinfo = a.w.kinfo + (size_t)lev * 4 * a.nmax;
  const int nr = kinfo[2 * slot + 1];
  const int* perm = a.w.perm + (size_t)lev * a.nmax + lo;
  const int* wpos = a.w.wpos + (size_t)lev * a.nmax + lo;
  const int* rotp = a.w.rotp + (size_t)lev * a.nmax + lo;
  const int* rotn = a.w.rotn + (size_t)lev * a.nmax + lo;
  const double* rotc = a.w.rotc + (size_t)lev * a.nmax + lo;
  const double* rots = a.w.rots + (size_t)lev * a.nmax + lo;
  double* tw = sm;
  for (int k = tid; k < m; k += DCB) tw[wpos[k]] = a.w.tk[lo + k];
  __syncthreads();
  if (tid == 0) {
    for (int t = nr - 1; t >= 0; --t) {
      const int pa = rotp[t], pb = rotn[t];
      const double c_ = rotc[t], s_ = rots[t];
      const double wa = tw[pa], wb = tw[pb];
      tw[pa] = c_ * wa - s_ * wb;
      tw[pb] = s_ * wa + c_ * wb;
    }
  }
  __syncthreads();
  for (int p = tid; p < m; p += DCB) a.w.tv[Pn][lo + perm[p]] = tw[p];
}

// ================================================== driver
// steps 1 and 2 (tridiagonalisation with b carried along, then the divide
// and conquer merges up to the root), shared by the solve and the spectrum
static int pinv_forward(int n, const double* T, const double* b, const PinvWs& w, int nmax,
                        double cutoff, uint32_t* status, hipStream_t s, DcArgs& da,
                        std::vector<size_t>& ubase) {
  // the partial sums of column norms (one per 64 rows) use merge scratch
  TriArgs ta{w.A, w.V, w.W, w.tau, w.d, w.e, w.bq, w.y, w.s12, w.col, w.pd, w.es, w.dl, w.scal, n};
  const size_t nn = (size_t)n * n;
  k_pinv_copy<<<(unsigned)((nn + 255) / 256), 256, 0, s>>>(T, w.A, nn, b, w.bq, n);
  MINSR_CHECK_LAUNCH();
  // 1. tridiagonalisation
  k_tri_row<0><<<(unsigned)((n + 63) / 64), 64, 0, s>>>(ta, -1, -1, 0);
  MINSR_CHECK_LAUNCH();
  for (int j0 = 0; j0 < n; j0 += TNB) {
    const int nb = std::min(TNB, n - j0);
    for (int p = 0; p < nb && j0 + p < n - 1; ++p) {
      const int j = j0 + p, rows = n - j - 1;
      const int rb = (j + 1) / (8 * TMR) * 8, nrow = (n + TMR - 1) / TMR - rb;
      k_tri_mv<<<(unsigned)(nrow + (2 * p + TMR - 1) / TMR), 64 * TMR, 0, s>>>(ta, j, p, rb, nrow,
                                                                               (rows + 64) / 64);
      MINSR_CHECK_LAUNCH();
      const unsigned grid = (unsigned)((rows + 63) / 64);
      const int npd = (n + TMR - 1) / TMR - (j + 1) / TMR;
      if (p == 0) k_tri_row<0><<<grid, 64, 0, s>>>(ta, j, p, npd);
      else if (p <= 4) k_tri_row<4><<<grid, 64, 0, s>>>(ta, j, p, npd);
      else if (p <= 8) k_tri_row<8><<<grid, 64, 0, s>>>(ta, j, p, npd);
      else k_tri_row<16><<<grid, 64, 0, s>>>(ta, j, p, npd);
      MINSR_CHECK_LAUNCH();
    }
    const int j1 = j0 + nb;
    if (j1 < n) {
      const unsigned tiles = (unsigned)((n - j1 + 63) / 64);
      k_tri_syr2k<<<dim3(tiles, tiles), 256, 0, s>>>(w.A, w.V, w.W, n, j1, nb);
      MINSR_CHECK_LAUNCH();
    }
  }
  // 2. divide and conquer, leaves at depth D
  const int D = depth_of(n);
  da = DcArgs{w, n, nmax, D, 0, 0, cutoff, status};
  k_dc_init<<<1, TBS, 0, s>>>(da);
  MINSR_CHECK_LAUNCH();
  ubase.assign(D + 1, 0);
  {
    size_t u = 0;
    for (int l = 0; l <= D; ++l) { ubase[l] = u; u += u_level_elems(n, l); }
  }
  for (int lev = D - 1; lev >= 0; --lev) {
    da.ubase = ubase[lev];
    const size_t mm = mmax_of(n, lev);
    da.umm = mm * mm;
    const unsigned nodes = 1u << lev;
    const size_t shm_prep = mm * 3 * sizeof(double);
    k_dc_rank<<<dim3((unsigned)((mm + 63) / 64), nodes), 64, mm * sizeof(double), s>>>(da, lev);
    MINSR_CHECK_LAUNCH();
    k_dc_prep<<<nodes, DCB, shm_prep, s>>>(da, lev);
    MINSR_CHECK_LAUNCH();
    k_dc_secular<<<dim3((unsigned)((mm + SEC_WAVES - 1) / SEC_WAVES), nodes), 64 * SEC_WAVES,
                   mm * 2 * sizeof(double), s>>>(da, lev);
    MINSR_CHECK_LAUNCH();
    k_dc_zhat<<<dim3((unsigned)((mm + 3) / 4), nodes), 256, 0, s>>>(da, lev);
    MINSR_CHECK_LAUNCH();
    k_dc_ucols<<<dim3((unsigned)((mm + 3) / 4), nodes), 256, 0, s>>>(da, lev);
    MINSR_CHECK_LAUNCH();
  }
  return MINSR_OK;
}

static int pinv_check(int n, const double* eig, size_t eig_elems, int nmax) {
  if (n > PINV_MAX_N)
    return fail(MINSR_E_UNSUPPORTED, "pseudo-inverse / spectrum: n = " + std::to_string(n) +
                                         " above " + std::to_string(PINV_MAX_N));
  if (!eig || eig_elems < pinv_workspace_doubles(nmax) || n > nmax)
    return fail(MINSR_E_INVALID_ARG, "pseudo-inverse workspace missing or too small");
  return MINSR_OK;
}

// the eigenvalues at the root (unscaled), in ascending order: position of
// entry i = number of entries below it, ties broken by index
__global__ __launch_bounds__(256) void k_eig_sorted(const double* ev, const double* scal, int n,
                                                    double* w) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const double v = ev[i];
  int r = 0;
  for (int j = 0; j < n; ++j) {
    const double u = ev[j];
    r += (u < v || (u == v && j < i)) ? 1 : 0;
  }
  w[r] = v * scal[0];
}

// App. E: (w_min, w_max, kappa_2(T + lambda I), d = -log10(kappa_2 eps)),
// T positive semidefinite (w_min taken as max(w_min, 0))
__global__ void k_condition(const double* w, int n, double lambda, double eps, double* cond) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double wmin = w[0], wmax = w[n - 1];
  const double den = fmax(wmin, 0.0) + lambda;
  const double k = den > 0.0 ? (wmax + lambda) / den : INFINITY;
  cond[0] = wmin;
  cond[1] = wmax;
  cond[2] = k;
  cond[3] = isfinite(k) ? -log10(k * eps) : -INFINITY;
}

int launch_spectrum(int n, const double* T, double lambda, double eps, double* w_out,
                    double* cond, double* eig, size_t eig_elems, int nmax, uint32_t* status,
                    hipStream_t s) {
  if (n == 0) return MINSR_OK;
  int rc = pinv_check(n, eig, eig_elems, nmax);
  if (rc) return rc;
  PinvWs w = carve(eig, n, nmax);
  DcArgs da{};
  std::vector<size_t> ubase;
  // the carried vector plays no part in the eigenvalues: the first row of T
  rc = pinv_forward(n, T, T, w, nmax, 0.0, status, s, da, ubase);
  if (rc) return rc;
  k_eig_sorted<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(w.ev[0], w.scal, n, w_out);
  MINSR_CHECK_LAUNCH();
  if (cond) {
    k_condition<<<1, 64, 0, s>>>(w_out, n, lambda, eps, cond);
    MINSR_CHECK_LAUNCH();
  }
  return MINSR_OK;
}

int launch_pinv_solve(int n, double* T, double cutoff, const double* b, double* x, double* eig,
                      size_t eig_elems, int nmax, uint32_t* status, hipStream_t s) {
  if (n == 0) return MINSR_OK;
  int rc = pinv_check(n, eig, eig_elems, nmax);
  if (rc) return rc;
  PinvWs w = carve(eig, n, nmax);
  DcArgs da{};
  std::vector<size_t> ubase;
  rc = pinv_forward(n, T, b, w, nmax, cutoff, status, s, da, ubase);
  if (rc) return rc;
  const int D = da.D;
  // 3. weights at the root, then down the tree
  k_dc_root<<<1, TBS, 0, s>>>(da);
  MINSR_CHECK_LAUNCH();
  for (int lev = 0; lev < D; ++lev) {
    da.ubase = ubase[lev];
    const size_t mm = mmax_of(n, lev);
    da.umm = mm * mm;
    const unsigned nodes = 1u << lev;
    k_dc_down_gemv<<<dim3((unsigned)((mm + 63) / 64), nodes), 256, 0, s>>>(da, lev);
    MINSR_CHECK_LAUNCH();
    k_dc_down_post<<<nodes, DCB, mm * sizeof(double), s>>>(da, lev);
    MINSR_CHECK_LAUNCH();
  }
  // 4. x = Q y
  const double* xin = w.tv[D & 1];
  const int blocks = (n + BKB - 1) / BKB;
  k_back_gram<<<dim3((unsigned)blocks, BKB / 16), 256, 0, s>>>(w.A, w.bg, n);
  MINSR_CHECK_LAUNCH();
  for (int b = blocks - 1; b >= 0; --b) {
    k_back_dot<<<BKB, 256, 0, s>>>(w.A, xin, w.sv, n, b * BKB);
    MINSR_CHECK_LAUNCH();
    k_back_upd<<<(unsigned)((n + 63) / 64), 64, 0, s>>>(w.A, w.tau, w.bg, w.sv, xin, x, n, b * BKB);
    MINSR_CHECK_LAUNCH();
    xin = x;
  }
  return MINSR_OK;
}

}  // namespace minsr
