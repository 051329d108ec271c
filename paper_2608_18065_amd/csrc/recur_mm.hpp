// The recurrence of gru.hip (Sec. 2, Eqs. 3-7; App. A) on the FP32 and FP64
// matrix cores: exact sampling, evaluation of given configurations, and (FP64,
// and FP32 2D) re-evaluation of Hamiltonian-connected configurations for local
// energies.
//
// Arithmetic.  v_mfma_f32_16x16x4_f32 and v_mfma_f64_16x16x4_f64 add their
// four products to the accumulator as a chain of fused multiply-adds in
// ascending k (compared with fma chains over 5e4 random tiles each on
// gfx950: all bits equal).  The accumulators start at the bias and input
// columns and take the inputs in k_forward's order, the cell and the head
// keep its expressions and the head's sums its tree, so every output here
// equals k_forward's bit for bit and either kernel may serve a call.
//
// Layout.  A workgroup advances 16 sequences; wave w owns hidden units
// 16w .. 16w + 15 and holds its rows of the gate weights (and of U1, U2)
// in registers for the whole kernel as A operands, so a site reads no
// weights (k_forward streams them from L2 for every one or two sequences:
// 328 KB a site at d_h = 128 in 2D, which bounds it).  States are the B
// operands: shared memory holds them as [unit % 4][sequence][unit / 4], so a
// lane reads the inputs of four (FP64: two) K-steps at once.  A lane of the
// result holds units 4 (lane / 16) .. + 3 of one sequence (the FP64 result
// rows are permuted to that by the choice of A rows): the cell runs in
// registers.  In 2D one state slot per lattice column is enough: at site
// (i, j) slot i still holds site (i, j - 1), the vertical predecessor, and is
// then overwritten.
//
// Measured: 10 x 10 sampling, d_h = 128, Ns = 4096 4161 -> 797 us (a site about
// 20k cycles, the products' issue 10k of them, the cells' about 5k); FP64 6 x 6
// local energies, d_h = 32, 251 samples 1352 -> 197 us.  FP32 2D local energies
// (RM_ELOC_SPLIT), 9 x 9, d_h = 128, 1024 samples 16.1 -> 7.9 ms against a
// kernel of 32 sequences and one wave a SIMD that streamed U1 | U2 from L2 and
// kept its window of states in global memory (56k cycles a site of 32, a third
// of them its work); here about 14k a site of 16 (products 5.5k).  FP64 7 x 6,
// d_h = 8, 256 samples: evaluation 133 -> 84 us, local energies 1082 -> 206.
#pragma once

#include <mutex>

#include "cell.hpp"
#include "mm.hpp"

namespace minsr {

// RM_ELOC_SPLIT: FP32 2D local energies with the gate products as FP16 hi/lo
// pairs and the hardware exp2 and reciprocal in the cell, both as the 1D local
// energies have them (gru_mfma.hip); the h' product stays FP32
enum { RM_SAMPLE = 0, RM_EVAL = 1, RM_ELOC = 2, RM_ELOC_SPLIT = 3 };

template <typename T> struct RecArgs {
  Work<T> w;
  int N, Lx, Ly, Ns, zero_mag, cplx, marshall, store_every;
  const double* uniforms;
  uint64_t key, counter;
  const uint64_t* counter_ptr;
  uint32_t* zero_word;
  const uint8_t* sigma_in;
  uint8_t* sigma_out;
  double* logpsi;          // optional [Ns][2]
  T* states;               // optional [Ns][N][H]
  T* gates;                // optional tape: 1D [Ns][N][4][H] u, r, candidate pre-activation,
                           // candidate; 2D [Ns][N][5][H], the cell input h' last
  double* site;            // optional [Ns][N][4]
  // local energies
  const T* states_in;
  const double* site_in;
  const uint8_t* subA;
  const int* bonds;
  const int* list;         // J1-J2: [M][Ns] samples with a nonzero matrix element
  const int* count;        //        their counts, then the number of items of 32
  const int* items;        //        [items][2] (term, chunk of 32 samples)
  int n_nn, ham_kind, M, nchunks;
  double hx, J1, J2;
  double* contrib;
};

// Sites whose conditionals one wave forms at once (head sums are kept for two
// batches).  Waiting for that wave once in four sites instead of at each takes
// 6 % off the 9 x 9 local energies and 5 x 5 evaluations (9.34 -> 8.81 ms); in
// the FP64 local energies the four-fold head sums cost a workgroup of the
// three a compute unit holds (7 x 6, d_h = 32: 407 -> 476 us).
template <typename T> constexpr int rec_batch(int mode) {
  return mode == RM_SAMPLE || (mode == RM_ELOC && sizeof(T) == 8) ? 1 : 4;
}

// bytes of shared memory of a workgroup
template <typename T> struct RecShape {
  static __host__ __device__ constexpr int slots(int dim, int Lx) { return dim == 1 ? 2 : Lx + 1; }
  static size_t bytes(int H, int dim, int Lx, int N, int mode) {
    const int ds = dim == 1 ? 2 : 4;
    const size_t t = (size_t)(3 * ds + 8) * H + mm_slot<T>(H) * slots(dim, Lx) +
                     (size_t)2 * rec_batch<T>(mode) * mm_tiles(H) * 64;
    return t * sizeof(T) + 16 * 4 * 8 + (size_t)16 * N + 64 + (3 * H + 16) * sizeof(float);
  }
};

template <typename T, int H, int DIM, int MODEX>
__global__ __launch_bounds__(64 * mm_tiles(H), sizeof(T) == 8 && H == 64 && DIM == 2 ? 1 : 2) void k_rec_mm(RecArgs<T> a) {
  using M = MM<T>;
  using acc_t = typename M::acc;
  using vec_t = typename M::vec;
  constexpr bool SPLIT = MODEX == RM_ELOC_SPLIT;
  constexpr int MODE = SPLIT ? RM_ELOC : MODEX;
  constexpr int NW = mm_tiles(H), NT = 64 * NW, KT = H / 4, V = M::V;
  constexpr int EU = mm_lane_units(H);
  constexpr int ds = DIM == 1 ? 2 : 4;
  constexpr int PT = mm_pitch<T>(H);
  constexpr size_t SLOT = mm_slot<T>(H);
  constexpr int CB = rec_batch<T>(MODE), PR = 2 * CB;   // sites settled at once, head sums kept
  extern __shared__ __align__(16) unsigned char rsm[];
  T* xc = reinterpret_cast<T*>(rsm);                 // [3][ds][H]
  T* bias = xc + 3 * ds * H;                         // [4][H]
  T* head = bias + 4 * H;                            // [4][H]
  T* X = head + 4 * H;                               // state slots
  const int nslot = RecShape<T>::slots(DIM, a.Lx);
  T* part = X + SLOT * nslot;                        // [PR][NW][16][4] head sums of the waves
  double* run = reinterpret_cast<double*>(part + PR * NW * 64);   // [16][4] running log-amplitudes
  uint8_t* spin = reinterpret_cast<uint8_t*>(run + 64);          // [N][16]
  T* XI = X + SLOT * a.Lx;                           // 2D: the cell input h' (split: [16][H + 4])
  float* sup = reinterpret_cast<float*>(spin + (((size_t)16 * a.N + 15) & ~(size_t)15));   // split: [3][H]
  float* hmx = sup + 3 * H;                          // weight row scales; [NW] largest |h'| of a wave

  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int n = l & 15, q = l >> 4;
  const int N = a.N, Lx = a.Lx;
  const int j0 = mm_first<H>(w, q);                  // this lane's units j0 .. j0 + EU - 1
  auto sync = [&]() { mm_sync<NW>(); };

  // which term and samples (local energies), or the 16 samples of the block
  int f1 = -1, f2 = -1, term = 0;
  double Jt = 0.0;
  int s = blockIdx.x * 16 + n;
  bool act = s < a.Ns;
  if constexpr (MODE == RM_ELOC) {
    int at;
    if (a.list) {
      const int it = blockIdx.x >> 1;
      if (it >= a.count[a.M]) return;                // uniform over the workgroup
      term = a.items[2 * it];
      at = 32 * a.items[2 * it + 1] + 16 * (blockIdx.x & 1);
      const int cnt = a.count[term];
      if (at >= cnt) return;                         // uniform
      f1 = a.bonds[2 * term]; f2 = a.bonds[2 * term + 1];
      Jt = term < a.n_nn ? a.J1 : a.J2;
      act = at + n < cnt;
      s = a.list[(size_t)term * a.Ns + min(at + n, cnt - 1)];
    } else {
      term = blockIdx.x / a.nchunks;
      s = 16 * (blockIdx.x % a.nchunks) + n;
      act = s < a.Ns;
      f1 = term;
    }
  }
  const int sid = MODE == RM_ELOC && a.list ? s : min(s, a.Ns - 1);
  const int k0 = f1;                                 // -1 outside local energies
  if constexpr (MODE == RM_SAMPLE)
    if (a.zero_word && blockIdx.x == 0 && tid == 0) a.zero_word[0] = 0u;

  // ---- set-up: constants and spins into shared memory
  for (int i = tid; i < 3 * ds * H; i += NT) xc[i] = a.w.xc[i];
  for (int i = tid; i < 4 * H; i += NT) { bias[i] = a.w.bias[i]; head[i] = a.w.head[i]; }
  const T c0 = a.w.headb[0], c1 = a.w.headb[1], cp0 = a.w.headb[2], cp1 = a.w.headb[3];
  if constexpr (MODE != RM_SAMPLE) {
    // lane group q of wave w reads every (4 NW)-th site of sequence n
    for (int k = 4 * w + q; k < N; k += 4 * NW) {
      int v = (int)(a.sigma_in[(size_t)sid * N + k] & 1);
      if (MODE == RM_ELOC && (k == f1 || k == f2)) v ^= 1;
      spin[16 * k + n] = (uint8_t)v;
    }
  }
  // A operands: row n of this wave's tile, input 4 t + q of step t
  const int jt = mm_unit<T, H>(w, n), ja = min(jt, H - 1);
  const bool arow = jt < H;
  constexpr int KF = H / 32;
  T wg[SPLIT ? 1 : 3][KT], wu[DIM == 2 ? 2 * KT : 1];
  mf16::h16x8 wh[SPLIT ? 3 : 1][SPLIT ? KF : 1], wl[SPLIT ? 3 : 1][SPLIT ? KF : 1];
  if constexpr (SPLIT) {
    // inputs 32 t + 8 q + e of row ja; a row reaching 2^14 is split as w 2^-s
    // and its products scaled back by 2^s (exact)
    auto wv = [&](int g, int i) { return a.w.fw[((size_t)(i >> 2) * H + ja) * 12 + g * 4 + (i & 3)]; };
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      float x[KF][8], mx = 0.f;
#pragma unroll
      for (int t = 0; t < KF; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          x[t][e] = wv(g, 32 * t + 8 * q + e);
          mx = fmaxf(mx, fabsf(x[t][e]));
        }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const int se = mx >= 16384.f ? min(ilogbf(mx) - 13, 120) : 0;
      const float dn = ldexpf(1.f, -se);
      if (q == 0) sup[g * H + ja] = ldexpf(1.f, se);
#pragma unroll
      for (int t = 0; t < KF; ++t) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[t][e] *= dn;
        mf16::split16(x[t], wh[g][t], wl[g][t]);
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const int k = 4 * t + q;
      const T* p = a.w.fw + ((size_t)(k / V) * H + ja) * 3 * V + k % V;
#pragma unroll
      for (int g = 0; g < 3; ++g) wg[g][t] = arow ? p[g * V] : (T)0;
    }
  }
  if constexpr (DIM == 2) {
    // U1 and U2 in k_forward's order: V inputs of U1, then the same of U2
#pragma unroll
    for (int t = 0; t < 2 * KT; ++t) {
      const int z = 4 * t + q, k = V * (z / (2 * V)) + z % V, u = (z / V) & 1;
      const T x = a.w.f2[((size_t)(k / V) * H + ja) * 2 * V + u * V + k % V];
      wu[t] = arow ? x : (T)0;
    }
  }

  // states the walk starts from
  T hp[EU] = {};                                     // 1D: the lane's units of h_{k-1}
  auto put = [&](T* slot, const T (&v)[EU]) {
#pragma unroll
    for (int e = 0; e < EU; ++e) slot[mm_place<T, H>(w, q, n, e)] = v[e];
  };
  const int kstart = k0 + 1;
  if constexpr (DIM == 1) {
    if (MODE == RM_ELOC) load4(a.states_in + ((size_t)sid * N + k0) * H + j0, hp);
    put(X + SLOT * (kstart & 1), hp);
  } else if constexpr (MODE == RM_ELOC) {
    // the latest site of the path up to k0 in every column
    const int jr = k0 / Lx;
    for (int i = 0; i < Lx; ++i) {
      int p = jr * Lx + ((jr & 1) ? Lx - 1 - i : i);
      if (p > k0) p = 2 * jr * Lx - 1 - p;           // the site above, if any
      T v[EU] = {};
      if (p >= 0) load4(a.states_in + ((size_t)sid * N + p) * H + j0, v);
      put(X + SLOT * i, v);
    }
  }
  if (tid < 64) run[tid] = 0.0;

  const int half = N / 2;
  int nup = 0, nA = 0, sp = -1;                       // nup: spins 0 up to the last settled site
  uint32_t cols = 0;                                 // 2D sampling: the latest spin of every column
  double mel = 0.0;
  int dA = 0;
  double lp = 0.0, ph = 0.0;
  const double* so = MODE == RM_ELOC ? a.site_in + (size_t)sid * N * 4 : nullptr;
  sync();
  if constexpr (MODE == RM_ELOC) {
    if (a.zero_mag)
      for (int k = 0; k <= k0; ++k) nup += spin[16 * k + n] == 0;
    const int vf = spin[16 * k0 + n];                // the flipped value
    sp = vf;
    if (w == 0 && q == 0) {
      // (new, old) log-probability and phase of the flipped site
      run[4 * n + 0] = so[4 * k0 + vf];
      run[4 * n + 1] = so[4 * k0 + 2 + vf];
      run[4 * n + 2] = 0.0 + so[4 * k0 + (vf ^ 1)];
      run[4 * n + 3] = 0.0 + so[4 * k0 + 2 + (vf ^ 1)];
    }
    auto old = [&](int k) -> int { return spin[16 * k + n] ^ ((k == f1 || k == f2) ? 1 : 0); };
    if (a.ham_kind == MINSR_HAM_TFIM) {
      mel = -a.hx;
    } else if (a.ham_kind == MINSR_HAM_CLUSTER) {
      mel = -(1.0 - 2.0 * old((f1 - 1 + N) % N)) * (1.0 - 2.0 * old((f1 + 1) % N));
    } else {
      mel = 0.5 * Jt;
    }
    if (a.marshall) {
      if (a.subA[f1]) dA += 1 - 2 * old(f1);
      if (f2 >= 0 && a.subA[f2]) dA += 1 - 2 * old(f2);
    }
    sync();
  }

  const uint64_t ctr = MODE == RM_SAMPLE ? (a.counter_ptr ? *a.counter_ptr : a.counter) : 0;
  U64x4 rw;
  rw.w[0] = rw.w[1] = rw.w[2] = rw.w[3] = 0;
  // log-conditionals and phases of site k from the waves' head sums, nu of
  // whose earlier spins are 0
  auto conditional = [&](int k, int nu, T& lp0, T& lp1, T& ph0, T& ph1) {
    const T* pb = part + (size_t)(k % PR) * NW * 64 + 4 * n;
    T z[4] = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c >= 2 && !a.cplx) continue;
      T v[NW];
#pragma unroll
      for (int i = 0; i < NW; ++i) v[i] = pb[i * 64 + c];
      if constexpr (NW == 1) z[c] = v[0];
      else if constexpr (NW == 2) z[c] = v[0] + v[1];
      else if constexpr (NW == 4) z[c] = (v[0] + v[1]) + (v[2] + v[3]);
      else z[c] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
    const T zz0 = z[0] + c0, zz1 = z[1] + c1;
    const T mx = zz0 > zz1 ? zz0 : zz1;
    const T d = zz0 > zz1 ? zz1 - zz0 : zz0 - zz1;   // -|z0 - z1|
    const T lse = mx + d_log1p(d_exp(d));
    lp0 = zz0 - lse;
    lp1 = zz1 - lse;
    if (a.zero_mag) {
      if (nu >= half) { lp0 = -INFINITY; lp1 = (T)0; }
      else if (k - nu >= half) { lp0 = (T)0; lp1 = -INFINITY; }
    }
    ph0 = ph1 = (T)0;
    if (a.cplx) {
      const T PI = (T)3.14159265358979323846;
      const T aa0 = z[2] + cp0, aa1 = z[3] + cp1;
      ph0 = PI * aa0 / ((T)1 + fabs(aa0));
      ph1 = PI * aa1 / ((T)1 + fabs(aa1));
    }
  };
  auto write_site = [&](int k, T lp0, T lp1, T ph0, T ph1) {
    double* st = a.site + ((size_t)s * N + k) * 4;
    st[0] = (double)lp0; st[1] = (double)lp1; st[2] = (double)ph0; st[3] = (double)ph1;
  };
  // sampling: the spin of site k, drawn in every lane of the sequence
  auto draw = [&](int k) {
    T lp0, lp1, ph0, ph1;
    conditional(k, nup, lp0, lp1, ph0, ph1);
    double u;
    if (a.uniforms) {
      u = a.uniforms[(size_t)sid * N + k];
    } else {
      // lane group g holds the Philox block of sites 4 g .. 4 g + 3 of
      // the current 16
      const int src = ((k >> 2) & 3) * 16 + n;
      const int c = k & 3;
      const uint64_t wq = c == 0 ? rw.w[0] : c == 1 ? rw.w[1] : c == 2 ? rw.w[2] : rw.w[3];
      u = u01(__shfl((unsigned long long)wq, src, 64));
    }
    const int v = u < (double)d_exp(lp0) ? 0 : 1;
    lp += (double)(v == 0 ? lp0 : lp1);
    ph += (double)(v == 0 ? ph0 : ph1);
    nup += v == 0;
    sp = v;
    if (w == 0 && q == 0 && act) {
      a.sigma_out[(size_t)s * N + k] = (uint8_t)v;
      if (a.site) write_site(k, lp0, lp1, ph0, ph1);
    }
  };
  // otherwise: sites kb .. kb + m - 1 (m <= CB) at once by one wave, lane group
  // q taking site kb + q; the running sums add the sites in order
  auto settle = [&](int kb, int m, double old_lp, double old_ph) {
    const int k = kb + min(q, m - 1);
    int nu = nup;
    if (a.zero_mag)
      for (int i = kb; i < k; ++i) nu += spin[16 * i + n] == 0;
    T lp0, lp1, ph0, ph1;
    conditional(k, nu, lp0, lp1, ph0, ph1);
    const int v = spin[16 * k + n];
    const double lpv = (double)(v == 0 ? lp0 : lp1), phv = (double)(v == 0 ? ph0 : ph1);
    double r[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) r[c] = run[4 * n + c];
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const int src = 16 * i + n;
      const double x0 = __shfl(lpv, src, 64), x1 = __shfl(phv, src, 64);
      if (i < m) { r[0] += x0; r[1] += x1; }
      if constexpr (MODE == RM_ELOC) {
        const double x2 = __shfl(old_lp, src, 64), x3 = __shfl(old_ph, src, 64);
        if (i < m) { r[2] += x2; r[3] += x3; }
      }
    }
    if (q == 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c) run[4 * n + c] = r[c];
    }
    if constexpr (MODE == RM_EVAL)
      if (a.site && act && q < m) write_site(k, lp0, lp1, ph0, ph1);
  };

  for (int k = kstart; k < N; ++k) {
    if constexpr (MODE == RM_SAMPLE)
      if (!a.uniforms && (k & 15) == 0)
        rw = philox4x64_10(ctr, (uint64_t)sid, (uint64_t)((k >> 2) + q), 0, a.key, 0);
    // the last site of a batch, and the wave that settles the batch
    const int kb = k - (k - kstart) % CB;
    const bool last = MODE != RM_SAMPLE && ((k - kstart) % CB == CB - 1 || k == N - 1);
    const bool mine = last && w == (k - kstart) / CB % NW;
    double old_lp = 0.0, old_ph = 0.0;
    if constexpr (MODE == RM_ELOC)
      if (mine) {
        // the sample's own conditionals, requested ahead of the site's work
        const int ks = min(kb + q, k);
        const int vo = spin[16 * ks + n] ^ (ks == f2 ? 1 : 0);
        old_lp = so[4 * ks + vo];
        old_ph = so[4 * ks + 2 + vo];
      }
    int sh = -1, sv = -1;
    T hin[EU];
    T* xin;
    T* out;
    if constexpr (DIM == 2) {
      const int j = k / Lx, kr = k - j * Lx;
      const int i = (j & 1) ? Lx - 1 - kr : kr;
      const bool hasH = kr > 0, hasV = j > 0;
      if constexpr (MODE == RM_SAMPLE) {
        if (hasH) sh = sp;
        if (hasV) sv = (int)(cols >> i) & 1;
      } else {
        if (hasH) sh = spin[16 * (k - 1) + n];
        if (hasV) sv = spin[16 * (2 * j * Lx - 1 - k) + n];
      }
      const T* xh = X + SLOT * ((j & 1) ? i + 1 : i - 1);
      const T* xv = X + SLOT * i;
      out = X + SLOT * i;
      xin = XI;
      // h' = U1 h_horizontal + U2 h_vertical
      acc_t acc = {(T)0, (T)0, (T)0, (T)0};
      if constexpr (V == 4) {
        const T* ph_ = xh + (q * 16 + n) * PT;
        const T* pv_ = xv + (q * 16 + n) * PT;
#pragma unroll
        for (int t4 = 0; t4 < KT / 4; ++t4) {
          T b1[4] = {(T)0, (T)0, (T)0, (T)0}, b2[4] = {(T)0, (T)0, (T)0, (T)0};
          if (hasH) load4(ph_ + 4 * t4, b1);
          if (hasV) load4(pv_ + 4 * t4, b2);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc = M::mma(wu[2 * (4 * t4 + e)], b1[e], acc);
            acc = M::mma(wu[2 * (4 * t4 + e) + 1], b2[e], acc);
          }
        }
      } else {
        // step t takes inputs 2 t, 2 t + 1 of both predecessors: lane groups
        // 0, 1 the horizontal one, 2, 3 the vertical one
        const bool has = q < 2 ? hasH : hasV;
        const T* p = (q < 2 ? xh : xv) + ((q & 1) * 16 + n) * PT;
#pragma unroll
        for (int m = 0; m < KT / 2; ++m) {
          double2 x = make_double2(0.0, 0.0), y = x;
          if (has) {
            x = *reinterpret_cast<const double2*>(p + 2 * m);
            y = *reinterpret_cast<const double2*>(p + 2 * 16 * PT + 2 * m);
          }
          acc = M::mma(wu[4 * m + 0], x.x, acc);
          acc = M::mma(wu[4 * m + 1], y.x, acc);
          acc = M::mma(wu[4 * m + 2], x.y, acc);
          acc = M::mma(wu[4 * m + 3], y.y, acc);
        }
      }
#pragma unroll
      for (int e = 0; e < EU; ++e) hin[e] = acc[e];
      if constexpr (SPLIT) {
        // h' is not bounded: the site's largest |h'| sets a power-of-two scale
        store4(XI + n * (H + 4) + j0, hin);
        float mx = fmaxf(fmaxf(fabsf(hin[0]), fabsf(hin[1])), fmaxf(fabsf(hin[2]), fabsf(hin[3])));
        mx = mf16::row16_max(mx);
        const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(r16[0]), __uint_as_float(r16[1]));
        const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(r32[0]), __uint_as_float(r32[1]));
        if (l == 0) hmx[w] = mx;
      } else {
        put(XI, hin);
      }
      sync();
    } else {
      sh = sp;
      xin = X + SLOT * (k & 1);
      out = X + SLOT * ((k + 1) & 1);
#pragma unroll
      for (int e = 0; e < EU; ++e) hin[e] = hp[e];
    }

    // gate pre-activations: bias and spin-input columns first
    acc_t ga[3] = {};
    T ai[EU];
    {
      T b[EU], x[EU];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        load4(bias + g * H + j0, b);
        const int gx = g < 2 ? g : 2;                // the candidate's input term is row 2
        if (g != 2) {
          if (sh >= 0) {
            load4(xc + (gx * ds + sh) * H + j0, x);
#pragma unroll
            for (int e = 0; e < EU; ++e) b[e] += x[e];
          }
          if (DIM == 2 && sv >= 0) {
            load4(xc + (gx * ds + (DIM == 2 ? 2 : 0) + sv) * H + j0, x);
#pragma unroll
            for (int e = 0; e < EU; ++e) b[e] += x[e];
          }
        }
#pragma unroll
        for (int e = 0; e < EU; ++e) {
          if (g < 3) ga[g][e] = b[e];
          else ai[e] = b[e];
        }
      }
    }
    if constexpr (SPLIT) {
      float mx = hmx[0];
#pragma unroll
      for (int i = 1; i < NW; ++i) mx = fmaxf(mx, hmx[i]);
      const int t2 = mx >= 16384.f ? min(ilogbf(mx) - 13, 120) : 0;
      const float hdn = ldexpf(1.f, -t2), hup = ldexpf(1.f, t2);
      const float* p = xin + n * (H + 4) + 8 * q;
      acc_t sa[3] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int t = 0; t < KF; ++t) {
        const float4 x0 = *reinterpret_cast<const float4*>(p + 32 * t);
        const float4 x1 = *reinterpret_cast<const float4*>(p + 32 * t + 4);
        const float x[8] = {x0.x * hdn, x0.y * hdn, x0.z * hdn, x0.w * hdn,
                            x1.x * hdn, x1.y * hdn, x1.z * hdn, x1.w * hdn};
        mf16::h16x8 bh, bl;
        mf16::split16(x, bh, bl);
#pragma unroll
        for (int g = 0; g < 3; ++g) sa[g] = mf16::mma16(wl[g][t], bh, sa[g]);
#pragma unroll
        for (int g = 0; g < 3; ++g) sa[g] = mf16::mma16(wh[g][t], bl, sa[g]);
#pragma unroll
        for (int g = 0; g < 3; ++g) sa[g] = mf16::mma16(wh[g][t], bh, sa[g]);
      }
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        float u[4];
        load4(sup + g * H + j0, u);
#pragma unroll
        for (int e = 0; e < 4; ++e) ga[g][e] = fmaf(sa[g][e], u[e] * hup, ga[g][e]);
      }
    } else {
      const T* p = xin + (q * 16 + n) * PT;
#pragma unroll
      for (int tv = 0; tv < KT / V; ++tv) {
        const vec_t x = *reinterpret_cast<const vec_t*>(p + V * tv);
        const T* xs = reinterpret_cast<const T*>(&x);
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
          for (int g = 0; g < 3; ++g) ga[g] = M::mma(wg[g][V * tv + e], xs[e], ga[g]);
      }
    }
    T hn[EU], gu[EU], gr[EU], ag[EU], gt[EU];
#pragma unroll
    for (int e = 0; e < EU; ++e) {
      ag[e] = ga[2][e];
      if constexpr (SPLIT) {
        gu[e] = mf16::sigm_hw(ga[0][e]);
        gr[e] = mf16::sigm_hw(ga[1][e]);
        gt[e] = mf16::tanh_hw(fmaf(gr[e], ag[e], ai[e]));
        hn[e] = ((T)1 - gu[e]) * hin[e] + gu[e] * gt[e];
        continue;
      }
      gu[e] = d_sigmoid(ga[0][e]);
      gr[e] = d_sigmoid(ga[1][e]);
      gt[e] = d_tanh(gr[e] * ag[e] + ai[e]);
      hn[e] = ((T)1 - gu[e]) * hin[e] + gu[e] * gt[e];
    }
    put(out, hn);
    // head: the lane's four units, the sequence's four lanes, the waves
    {
      T u[EU];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (c >= 2 && !a.cplx) continue;
        load4(head + c * H + j0, u);
        T z = u[0] * hn[0] + u[1] * hn[1];
        if constexpr (EU == 4) z = z + (u[2] * hn[2] + u[3] * hn[3]);
        z = xor32_sum(xor16_sum(z));
        if (q == 0) part[((size_t)(k % PR) * NW + w) * 64 + 4 * n + c] = z;
      }
    }
    if constexpr (MODE != RM_ELOC) {
      if (act) {
        const size_t row = (size_t)s * N + k;
        if (a.states && (DIM == 2 || (k + 1) % a.store_every == 0))
          store4(a.states + row * H + j0, hn);
        if (a.gates) {
          T* g = a.gates + row * (DIM == 1 ? 4 : 5) * H + j0;
          store4(g, gu); store4(g + H, gr); store4(g + 2 * H, ag); store4(g + 3 * H, gt);
          if constexpr (DIM == 2) store4(g + 4 * H, hin);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < EU; ++e) hp[e] = hn[e];
    sync();
    const int jr = k / Lx, ir = (jr & 1) ? Lx - 1 - (k - jr * Lx) : k - jr * Lx;
    if constexpr (MODE == RM_SAMPLE) {
      draw(k);
      if (a.marshall && !((ir + jr) & 1)) nA += sp;
      if constexpr (DIM == 2) cols = (cols & ~(1u << ir)) | ((uint32_t)sp << ir);
    } else {
      if (mine) settle(kb, k - kb + 1, old_lp, old_ph);
      if (DIM == 1) sp = spin[16 * k + n];
      if (a.zero_mag && last)
        for (int i = kb; i <= k; ++i) nup += spin[16 * i + n] == 0;
      if constexpr (MODE == RM_EVAL)
        if (a.marshall && !((ir + jr) & 1)) nA += spin[16 * k + n];
    }
  }
  if constexpr (MODE != RM_SAMPLE) {
    sync();
    lp = run[4 * n];
    ph = run[4 * n + 1];
  }
  if (w != 0 || q != 0 || !act) return;
  if constexpr (MODE == RM_ELOC) {
    const double dre = 0.5 * (lp - run[4 * n + 2]);
    const double dim_ = (ph - run[4 * n + 3]) + 3.14159265358979323846 * (double)dA;
    const double e = mel == 0.0 ? 0.0 : exp(dre);
    double* o = a.contrib + ((size_t)term * a.Ns + s) * 2;
    o[0] = mel * e * cos(dim_);
    o[1] = mel * e * sin(dim_);
  } else if (a.logpsi) {
    a.logpsi[2 * s] = 0.5 * lp;
    a.logpsi[2 * s + 1] = ph + 3.14159265358979323846 * (double)nA;
  }
}

// shared memory of the launch (whether a call may take the kernel)
template <typename T>
static size_t rec_smem(const minsr_model* m, int mode) {
  return RecShape<T>::bytes(m->H, m->dim, m->d.Lx, m->N, mode);
}

template <typename T>
static bool rec_fits(const minsr_model* m) {
  return !m->linear && m->H >= (sizeof(T) == 4 ? 16 : 8) && m->H <= (sizeof(T) == 4 ? 128 : 64) &&
         rec_smem<T>(m, RM_EVAL) <= MM_LDS;   // the largest of the modes
}

template <typename T, int H, int DIM, int MODE>
static int rec_launch(const RecArgs<T>& a, unsigned grid, size_t smem, hipStream_t s) {
  // more than 64 KiB of dynamic shared memory: allowed once per process
  static std::once_flag once;
  hipError_t attr = hipSuccess;
  std::call_once(once, [&] {
    attr = hipFuncSetAttribute((const void*)k_rec_mm<T, H, DIM, MODE>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)MM_LDS);
  });
  MINSR_HIP(attr);
  k_rec_mm<T, H, DIM, MODE><<<grid, 64 * mm_tiles(H), smem, s>>>(a);
  MINSR_CHECK_LAUNCH();
  return MINSR_OK;
}

template <typename T, int MODE>
static int rec_dispatch(const minsr_model* m, const RecArgs<T>& a, unsigned grid, hipStream_t s) {
  const size_t smem = rec_smem<T>(m, MODE);
  if (m->dim == 1) {
    switch (m->H) {
      case 8: if constexpr (sizeof(T) == 8) return rec_launch<T, 8, 1, MODE>(a, grid, smem, s); break;
      case 16: return rec_launch<T, 16, 1, MODE>(a, grid, smem, s);
      case 32: return rec_launch<T, 32, 1, MODE>(a, grid, smem, s);
      case 64: return rec_launch<T, 64, 1, MODE>(a, grid, smem, s);
      case 128: if constexpr (sizeof(T) == 4) return rec_launch<T, 128, 1, MODE>(a, grid, smem, s);
    }
  } else {
    switch (m->H) {
      case 8: if constexpr (sizeof(T) == 8) return rec_launch<T, 8, 2, MODE>(a, grid, smem, s); break;
      case 16: return rec_launch<T, 16, 2, MODE>(a, grid, smem, s);
      case 32: return rec_launch<T, 32, 2, MODE>(a, grid, smem, s);
      case 64: return rec_launch<T, 64, 2, MODE>(a, grid, smem, s);
      case 128: if constexpr (sizeof(T) == 4) return rec_launch<T, 128, 2, MODE>(a, grid, smem, s);
    }
  }
  return fail(MINSR_E_UNSUPPORTED, "matrix-core recurrence: hidden width");
}

template <typename T>
static RecArgs<T> rec_args(const minsr_model* m, const Work<T>& w, int Ns) {
  RecArgs<T> a{};
  a.w = w;
  a.N = m->N; a.Lx = m->d.Lx; a.Ly = m->d.Ly; a.Ns = Ns;
  a.zero_mag = m->d.zero_mag; a.cplx = m->cplx; a.marshall = m->d.marshall;
  a.store_every = 1;
  a.subA = m->subA;
  return a;
}

template <typename T>
static int rec_forward(minsr_model* m, const Work<T>& w, int mode, const RecCall& c,
                       hipStream_t s) {
  RecArgs<T> a = rec_args<T>(m, w, c.Ns);
  a.uniforms = c.uniforms; a.key = c.key; a.counter = c.counter; a.counter_ptr = c.counter_ptr;
  a.zero_word = c.zero_word;
  a.sigma_in = c.sigma; a.sigma_out = c.sigma;
  a.logpsi = c.logpsi; a.states = (T*)c.states; a.store_every = c.store_every;
  a.gates = c.store_every == 1 && c.Ns <= m->gates_ns ? (T*)c.gates : nullptr;
  a.site = c.site;
  const unsigned grid = (unsigned)((c.Ns + 15) / 16);
  return mode == 0 ? rec_dispatch<T, RM_SAMPLE>(m, a, grid, s)
                   : rec_dispatch<T, RM_EVAL>(m, a, grid, s);
}

template <typename T>
static int rec_eloc(minsr_model* m, const Work<T>& w, const minsr_hamiltonian* H, int Ns,
                    const uint8_t* sigma, const void* states, const double* site, int M,
                    hipStream_t s) {
  RecArgs<T> a = rec_args<T>(m, w, Ns);
  a.sigma_in = sigma; a.states_in = (const T*)states; a.site_in = site;
  a.bonds = m->bonds; a.n_nn = m->n_nn; a.ham_kind = H->kind; a.M = M;
  a.hx = H->h; a.J1 = H->J; a.J2 = H->J2; a.contrib = m->contrib;
  a.nchunks = (Ns + 15) / 16;
  unsigned grid = (unsigned)(a.nchunks * M);
  if (H->kind == MINSR_HAM_J1J2) {
    const int rc = launch_eloc_lists(m, Ns, sigma, M, s);
    if (rc) return rc;
    a.list = m->elist; a.count = m->ecount; a.items = m->eitems;
    grid = 2u * (unsigned)((Ns + 31) / 32) * (unsigned)M;   // at most; the rest leave at once
  }
  if constexpr (sizeof(T) == 4) {
    const size_t smem = rec_smem<T>(m, RM_ELOC_SPLIT);
    switch (m->H) {
      case 16: return m->dim == 1 ? rec_launch<T, 16, 1, RM_ELOC>(a, grid, smem, s)
                                  : rec_launch<T, 16, 2, RM_ELOC>(a, grid, smem, s);
      case 32: return rec_launch<T, 32, 2, RM_ELOC_SPLIT>(a, grid, smem, s);
      case 64: return rec_launch<T, 64, 2, RM_ELOC_SPLIT>(a, grid, smem, s);
      case 128: return rec_launch<T, 128, 2, RM_ELOC_SPLIT>(a, grid, smem, s);
    }
    return fail(MINSR_E_UNSUPPORTED, "matrix-core local energies: hidden width");
  } else {
    return rec_dispatch<T, RM_ELOC>(m, a, grid, s);
  }
}

}  // namespace minsr
