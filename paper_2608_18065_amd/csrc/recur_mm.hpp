// The recurrence of gru.hip (Sec. 2, Eqs. 3-7; App. A) on the FP32 and FP64
// matrix cores: exact sampling, evaluation of given configurations, and (FP64)
// re-evaluation of Hamiltonian-connected configurations for local energies.
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
#pragma once

#include <mutex>

#include "cell.hpp"
#include "mm.hpp"

namespace minsr {

namespace {

__device__ inline float xor16_sum(float v) { return mf16::sum_xor16(v); }
__device__ inline float xor32_sum(float v) { return mf16::sum_xor32(v); }
// both halves of a double through the VALU lane swap, as sum_xor16 / sum_xor32
template <bool ROW> __device__ inline double swap_sum(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
  const auto rl = ROW ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                      : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto rh = ROW ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                      : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  auto d = [](uint32_t l, uint32_t h) {
    return __longlong_as_double((long long)(((unsigned long long)h << 32) | l));
  };
  return d(rl[0], rh[0]) + d(rl[1], rh[1]);
}
__device__ inline double xor16_sum(double v) { return swap_sum<true>(v); }
__device__ inline double xor32_sum(double v) { return swap_sum<false>(v); }

}  // namespace

enum { RM_SAMPLE = 0, RM_EVAL = 1, RM_ELOC = 2 };

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

// bytes of shared memory of a workgroup
template <typename T> struct RecShape {
  static __host__ __device__ constexpr int slots(int dim, int Lx) { return dim == 1 ? 2 : Lx + 1; }
  static size_t bytes(int H, int dim, int Lx, int N) {
    const int ds = dim == 1 ? 2 : 4;
    const size_t t = (size_t)(3 * ds + 8) * H + mm_slot<T>(H) * slots(dim, Lx) +
                     (size_t)2 * (H / 16) * 64;
    return t * sizeof(T) + 16 * 4 * 8 + (size_t)16 * N + 64;
  }
};

template <typename T, int H, int DIM, int MODE>
__global__ __launch_bounds__(4 * H, sizeof(T) == 8 && H == 64 && DIM == 2 ? 1 : 2) void k_rec_mm(RecArgs<T> a) {
  using M = MM<T>;
  using acc_t = typename M::acc;
  using vec_t = typename M::vec;
  constexpr int NW = H / 16, NT = 64 * NW, KT = H / 4, V = M::V;
  constexpr int ds = DIM == 1 ? 2 : 4;
  constexpr int PT = mm_pitch<T>(H);
  constexpr size_t SLOT = mm_slot<T>(H);
  extern __shared__ __align__(16) unsigned char rsm[];
  T* xc = reinterpret_cast<T*>(rsm);                 // [3][ds][H]
  T* bias = xc + 3 * ds * H;                         // [4][H]
  T* head = bias + 4 * H;                            // [4][H]
  T* X = head + 4 * H;                               // state slots
  const int nslot = RecShape<T>::slots(DIM, a.Lx);
  T* part = X + SLOT * nslot;                        // [2][NW][16][4] head sums of the waves
  double* run = reinterpret_cast<double*>(part + 2 * NW * 64);   // [16][4] running log-amplitudes
  uint8_t* spin = reinterpret_cast<uint8_t*>(run + 64);          // [N][16]
  T* XI = X + SLOT * a.Lx;                           // 2D: the cell input h'

  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int n = l & 15, q = l >> 4;
  const int N = a.N, Lx = a.Lx;
  const int j0 = 16 * w + 4 * q;                     // this lane's units j0 .. j0 + 3
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
  const int ja = 16 * w + M::row(n);
  T wg[3][KT], wu[DIM == 2 ? 2 * KT : 1];
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    const int k = 4 * t + q;
    const T* p = a.w.fw + ((size_t)(k / V) * H + ja) * 3 * V + k % V;
#pragma unroll
    for (int g = 0; g < 3; ++g) wg[g][t] = p[g * V];
  }
  if constexpr (DIM == 2) {
    // U1 and U2 in k_forward's order: V inputs of U1, then the same of U2
#pragma unroll
    for (int t = 0; t < 2 * KT; ++t) {
      const int z = 4 * t + q, k = V * (z / (2 * V)) + z % V, u = (z / V) & 1;
      wu[t] = a.w.f2[((size_t)(k / V) * H + ja) * 2 * V + u * V + k % V];
    }
  }

  // states the walk starts from
  T hp[4] = {(T)0, (T)0, (T)0, (T)0};                // 1D: the lane's units of h_{k-1}
  auto put = [&](T* slot, const T (&v)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) slot[(e * 16 + n) * PT + 4 * w + q] = v[e];
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
      T v[4] = {(T)0, (T)0, (T)0, (T)0};
      if (p >= 0) load4(a.states_in + ((size_t)sid * N + p) * H + j0, v);
      put(X + SLOT * i, v);
    }
  }
  if (tid < 64) run[tid] = 0.0;

  const int half = N / 2;
  int nup = 0, ndn = 0, nA = 0, sp = -1;
  uint32_t cols = 0;                                 // 2D sampling: the latest spin of every column
  double mel = 0.0;
  int dA = 0;
  double lp = 0.0, ph = 0.0;
  const double* so = MODE == RM_ELOC ? a.site_in + (size_t)sid * N * 4 : nullptr;
  sync();
  if constexpr (MODE == RM_ELOC) {
    if (a.zero_mag)
      for (int k = 0; k <= k0; ++k) { const int v = spin[16 * k + n]; nup += v == 0; ndn += v == 1; }
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
  // conditional of site k from the head sums; sampling draws its spin in
  // every lane of the sequence, otherwise one wave keeps the running sums
  auto conditional = [&](int k, double old_lp, double old_ph) {
    const T* pb = part + (size_t)(k & 1) * NW * 64 + 4 * n;
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
    T lp0 = zz0 - lse, lp1 = zz1 - lse;
    if (a.zero_mag) {
      if (nup >= half) { lp0 = -INFINITY; lp1 = (T)0; }
      else if (ndn >= half) { lp0 = (T)0; lp1 = -INFINITY; }
    }
    T ph0 = (T)0, ph1 = (T)0;
    if (a.cplx) {
      const T PI = (T)3.14159265358979323846;
      const T aa0 = z[2] + cp0, aa1 = z[3] + cp1;
      ph0 = PI * aa0 / ((T)1 + fabs(aa0));
      ph1 = PI * aa1 / ((T)1 + fabs(aa1));
    }
    int v;
    if constexpr (MODE == RM_SAMPLE) {
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
      v = u < (double)d_exp(lp0) ? 0 : 1;
    } else {
      v = spin[16 * k + n];
    }
    const double lpv = (double)(v == 0 ? lp0 : lp1), phv = (double)(v == 0 ? ph0 : ph1);
    if constexpr (MODE == RM_SAMPLE) {
      lp += lpv; ph += phv;
      nup += v == 0; ndn += v == 1;
      if (w == 0 && q == 0 && act) a.sigma_out[(size_t)s * N + k] = (uint8_t)v;
      sp = v;
    } else if (q == 0) {
      run[4 * n] += lpv;
      run[4 * n + 1] += phv;
      if constexpr (MODE == RM_ELOC) {
        run[4 * n + 2] += old_lp;
        run[4 * n + 3] += old_ph;
      }
    }
    if constexpr (MODE != RM_ELOC)
      if (a.site && w == (MODE == RM_SAMPLE ? 0 : k % NW) && q == 0 && act) {
        double* st = a.site + ((size_t)s * N + k) * 4;
        st[0] = (double)lp0; st[1] = (double)lp1; st[2] = (double)ph0; st[3] = (double)ph1;
      }
  };

  for (int k = kstart; k < N; ++k) {
    if constexpr (MODE == RM_SAMPLE)
      if (!a.uniforms && (k & 15) == 0)
        rw = philox4x64_10(ctr, (uint64_t)sid, (uint64_t)((k >> 2) + q), 0, a.key, 0);
    double old_lp = 0.0, old_ph = 0.0;
    if constexpr (MODE == RM_ELOC)
      if (w == k % NW) {
        // the sample's own conditional, requested ahead of the site's work
        const int vo = spin[16 * k + n] ^ (k == f2 ? 1 : 0);
        old_lp = so[4 * k + vo];
        old_ph = so[4 * k + 2 + vo];
      }
    int sh = -1, sv = -1;
    T hin[4];
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
      for (int e = 0; e < 4; ++e) hin[e] = acc[e];
      put(XI, hin);
      sync();
    } else {
      sh = sp;
      xin = X + SLOT * (k & 1);
      out = X + SLOT * ((k + 1) & 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) hin[e] = hp[e];
    }

    // gate pre-activations: bias and spin-input columns first
    acc_t ga[3];
    T ai[4];
    {
      T b[4], x[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        load4(bias + g * H + j0, b);
        const int gx = g < 2 ? g : 2;                // the candidate's input term is row 2
        if (g != 2) {
          if (sh >= 0) {
            load4(xc + (gx * ds + sh) * H + j0, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] += x[e];
          }
          if (DIM == 2 && sv >= 0) {
            load4(xc + (gx * ds + (DIM == 2 ? 2 : 0) + sv) * H + j0, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] += x[e];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (g < 3) ga[g][e] = b[e];
          else ai[e] = b[e];
        }
      }
    }
    {
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
    T hn[4], gu[4], gr[4], ag[4], gt[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ag[e] = ga[2][e];
      gu[e] = d_sigmoid(ga[0][e]);
      gr[e] = d_sigmoid(ga[1][e]);
      gt[e] = d_tanh(gr[e] * ag[e] + ai[e]);
      hn[e] = ((T)1 - gu[e]) * hin[e] + gu[e] * gt[e];
    }
    put(out, hn);
    // head: the lane's four units, the sequence's four lanes, the waves
    {
      T u[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (c >= 2 && !a.cplx) continue;
        load4(head + c * H + j0, u);
        T z = (u[0] * hn[0] + u[1] * hn[1]) + (u[2] * hn[2] + u[3] * hn[3]);
        z = xor32_sum(xor16_sum(z));
        if (q == 0) part[((size_t)(k & 1) * NW + w) * 64 + 4 * n + c] = z;
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
    for (int e = 0; e < 4; ++e) hp[e] = hn[e];
    sync();
    if constexpr (MODE == RM_SAMPLE) {
      conditional(k, 0.0, 0.0);
      const int j = k / Lx, i = (j & 1) ? Lx - 1 - (k - j * Lx) : k - j * Lx;
      if (a.marshall && !((i + j) & 1)) nA += sp;
      if constexpr (DIM == 2) cols = (cols & ~(1u << i)) | ((uint32_t)sp << i);
    } else {
      if (w == k % NW) conditional(k, old_lp, old_ph);
      if (DIM == 1) sp = spin[16 * k + n];
      if (a.zero_mag) { const int v = spin[16 * k + n]; nup += v == 0; ndn += v == 1; }
      if constexpr (MODE == RM_EVAL) {
        const int j = k / Lx, i = (j & 1) ? Lx - 1 - (k - j * Lx) : k - j * Lx;
        if (a.marshall && !((i + j) & 1)) nA += spin[16 * k + n];
      }
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
static size_t rec_smem(const minsr_model* m) {
  return RecShape<T>::bytes(m->H, m->dim, m->d.Lx, m->N);
}

template <typename T>
static bool rec_fits(const minsr_model* m) {
  return !m->linear && m->H >= 16 && m->H <= (sizeof(T) == 4 ? 128 : 64) &&
         rec_smem<T>(m) <= MM_LDS;
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
  k_rec_mm<T, H, DIM, MODE><<<grid, 4 * H, smem, s>>>(a);
  MINSR_CHECK_LAUNCH();
  return MINSR_OK;
}

template <typename T, int MODE>
static int rec_dispatch(const minsr_model* m, const RecArgs<T>& a, unsigned grid, hipStream_t s) {
  const size_t smem = rec_smem<T>(m);
  if (m->dim == 1) {
    switch (m->H) {
      case 16: return rec_launch<T, 16, 1, MODE>(a, grid, smem, s);
      case 32: return rec_launch<T, 32, 1, MODE>(a, grid, smem, s);
      case 64: return rec_launch<T, 64, 1, MODE>(a, grid, smem, s);
      case 128: if constexpr (sizeof(T) == 4) return rec_launch<T, 128, 1, MODE>(a, grid, smem, s);
    }
  } else {
    switch (m->H) {
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

}  // namespace minsr
