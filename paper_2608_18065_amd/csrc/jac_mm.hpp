// Per-sample log-derivatives (Sec. 2.3, Alg. 1 step 5; the cell of App. A) on
// the FP32 and FP64 matrix cores, for the models whose forward pass leaves a
// tape of every site (2D models; FP64 chains): three launches per chunk of
// samples, equal to k_jacobian's rows bit for bit in FP32.
//
// k_jacobian gives every sample a workgroup that streams the gate weights and
// their transposes from L2 at each site and keeps the whole gradient in
// registers (10 x 10, d_h = 128, Ns = 4096: 42 ms for 1.4 GB of rows, bound by
// those streams).  Here
//   k_jac_head    forms the output head's conditionals of every site, 64 at a
//                 time per wave, with k_jacobian's reduction order;
//   k_jac_rev_mm  walks 16 rows at once backwards, with the transposed weights
//                 in registers as MFMA operands (recur_mm.hpp has the layout): a
//                 site is one [d_h x 3 d_h] x [3 d_h x 16] product for the cell
//                 input's adjoint and, in 2D, one [2 d_h x d_h] x [d_h x 16]
//                 product for the predecessors'; it writes the site's gate
//                 adjoints;
//   k_jac_rows_mm one workgroup per row: the weight blocks as [d_h x N] x
//                 [N x d_h] products over the sites, the rest as sums.
// The MFMAs add their products as ascending fma chains, so the order of
// k_jacobian's sums is kept by the order of the operands: the reverse product
// as its partial sums (4 per part of the rows), the weight blocks from the
// last site to the first.
//
// 10 x 10, d_h = 128, Ns = 4096 FP32: head 0.09 ms, reverse pass 0.93 (its
// products' issue 0.42, two barriers and the tape's latency a site with one
// workgroup a compute unit most of the rest), rows 1.34 (products 0.48; 3.3 GB
// read and 1.4 written), against 42.0 in k_jacobian.  It wins at every size:
// 7 x 6, Ns = 33: d_h = 32 0.25 / 0.45 ms with the evaluation, d_h = 64 0.43 /
// 1.11, d_h = 128 0.82 / 2.02; FP64 chain of 40, Ns = 33: d_h = 16 0.19 / 0.42,
// d_h = 64 0.46 / 1.35.  FP64 d_h = 8, 256 samples: 7 x 6 0.16 / 0.45, chain of
// 40 0.11 / 0.33.
#pragma once

#include <cmath>
#include <mutex>

#include "cell.hpp"
#include "mm.hpp"

namespace minsr {

template <typename T> struct JmArgs {
  Work<T> w;
  Layout L;
  int N, Lx, Ns, zero_mag, cplx;
  int s_base, ns;          // this chunk: samples [s_base, s_base + ns)
  const uint8_t* sigma;    // [Ns][N]
  const T* states;         // [Ns][N][H]
  const T* tape;           // [ns][N][4 or 5][H] of the chunk
  T* head;                 // [ns][N][4]: p0, p1, phase pre-activations a0, a1
  T* adj;                  // [seeds][ns][N][4 or 5][H]: adjoints of the u, r pre-activations,
                           // of W_h x + b_h, of the candidate's pre-activation, of x = h' (2D)
  T* O;                    // [seeds Ns][Np]
  T scale;
};

// ------------------------------------------------------------ output head
// one wave per PW (sample, site) pairs: per pair the sums over the units as
// k_jacobian forms them (an xor butterfly over 64 lanes, then the two
// wavefronts' halves at d_h = 128), then lane i the conditional of pair i.
// PW is 64, or 16 where that leaves SIMDs idle (640 pairs, d_h = 16: 12.9 ->
// 5.2 us).  The sums stay on the VALU and eight states are requested
// together: 10 x 10, d_h = 128, 4096 samples 153 -> 94 us.
template <typename T, int H, int PW>
__global__ __launch_bounds__(256) void k_jac_head(JmArgs<T> a) {
  constexpr int W = H < 64 ? H : 64, G = H / W;
  constexpr int PP = 64 / W;              // pairs side by side in a wave
  const int lane = threadIdx.x & 63;
  const long long p0 = PW * (4ll * blockIdx.x + (threadIdx.x >> 6));
  const long long np = (long long)a.ns * a.N;
  if (p0 >= np) return;                   // uniform per wave
  const int j = lane % W, sub = lane / W;
  const int nq = a.cplx ? 4 : 2;
  T u[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int c = 0; c < 4; ++c) u[g][c] = c < nq ? a.w.head[c * H + g * W + j] : (T)0;
  const T* st = a.states + (size_t)a.s_base * a.N * H;
  T z[4] = {(T)0, (T)0, (T)0, (T)0};
  constexpr int B = PW / PP < 8 ? PW / PP : 8;   // states requested together
  for (int i0 = 0; i0 < PW; i0 += PP * B) {
    T h[B][G];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const long long p = min(p0 + i0 + PP * b + sub, np - 1);
#pragma unroll
      for (int g = 0; g < G; ++g) h[b][g] = st[(size_t)p * H + g * W + j];
    }
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (c >= nq) continue;
        T t = (T)0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const T v = unit_sum<W>(u[g][c] * h[b][g]);
          t = g == 0 ? v : t + v;
        }
        // pair i0 + PP b + k's sum is in lanes k W ..; that lane keeps it
        const int at = lane - (i0 + PP * b);
        const T s0 = wave_lane<0>(t);
        if (at == 0) z[c] = s0;
        if constexpr (PP >= 2) { const T v = wave_lane<W % 64>(t); if (at == 1) z[c] = v; }
        if constexpr (PP >= 4) {
          const T v2 = wave_lane<2 * W % 64>(t), v3 = wave_lane<3 * W % 64>(t);
          if (at == 2) z[c] = v2;
          if (at == 3) z[c] = v3;
        }
        if constexpr (PP >= 8) {
          const T v4 = wave_lane<4 * W % 64>(t), v5 = wave_lane<5 * W % 64>(t);
          const T v6 = wave_lane<6 * W % 64>(t), v7 = wave_lane<7 * W % 64>(t);
          if (at == 4) z[c] = v4;
          if (at == 5) z[c] = v5;
          if (at == 6) z[c] = v6;
          if (at == 7) z[c] = v7;
        }
      }
  }
  const long long p = p0 + lane;
  if (lane >= PW || p >= np) return;
  const int N = a.N, k = (int)(p % N);
  const long long sl = p / N;
  const T zz0 = z[0] + a.w.headb[0], zz1 = z[1] + a.w.headb[1];
  const T mx = zz0 > zz1 ? zz0 : zz1;
  const T d = zz0 > zz1 ? zz1 - zz0 : zz0 - zz1;
  const T lse = mx + d_log1p(d_exp(d));
  T q0 = d_exp(zz0 - lse), q1 = d_exp(zz1 - lse);
  if (a.zero_mag) {
    const uint8_t* sg = a.sigma + (size_t)(a.s_base + sl) * N;
    int cu = 0;
    for (int i = 0; i < k; ++i) cu += (sg[i] & 1) == 0;
    if (cu >= N / 2) { q0 = (T)0; q1 = (T)1; }
    else if (k - cu >= N / 2) { q0 = (T)1; q1 = (T)0; }
  }
  const T o[4] = {q0, q1, z[2] + a.w.headb[2], z[3] + a.w.headb[3]};
  store4(a.head + 4 * p, o);
}

// adjoints of the two outputs of a site's head for one seed
template <typename T>
__device__ inline void head_adjoint(int seed, int sk, const T (&hd)[4], T& dz0, T& dz1) {
  if (seed == 0) {
    dz0 = (T)0.5 * ((sk == 0 ? (T)1 : (T)0) - hd[0]);
    dz1 = (T)0.5 * ((sk == 1 ? (T)1 : (T)0) - hd[1]);
  } else {
    const T PI = (T)3.14159265358979323846;
    const T e0 = (T)1 + fabs(hd[2]), e1 = (T)1 + fabs(hd[3]);
    dz0 = sk == 0 ? PI / (e0 * e0) : (T)0;
    dz1 = sk == 1 ? PI / (e1 * e1) : (T)0;
  }
}

// ------------------------------------------------------------ reverse pass
// Order of the reverse product's 3 H inputs (gate, i): the rows i are dealt in
// groups of V to NC = 4 P chains (part of the rows, group mod 4; d_h = 8: two
// a part); inside a
// group i runs over its V rows with the gates innermost.  Input e of chain c
// is element e % 4 of K-step (e / 4) NC + c, so that consecutive products
// belong to different chains.
template <typename T, int H, int P> struct RevOrder {
  static constexpr int V = MM<T>::V, CP = H < 16 ? 2 : 4, NC = CP * P, NS = 3 * H / (4 * NC);
  static constexpr int PITCH = 3 * H / 4 + V;
  static_assert(NS * 4 * NC == 3 * H && NS >= 1, "whole K-steps per chain");
  __device__ static void slot(int g, int i, int& step, int& el) {
    const int i4 = i / V, p = i4 / (H / P / V);
    const int within = (i4 - p * (H / P / V)) / CP;
    const int e = within * 3 * V + 3 * (i % V) + g;
    step = (e / 4) * NC + CP * p + i4 % CP;
    el = e & 3;
  }
  __device__ static void input(int step, int el, int& g, int& i) {
    const int c = step % NC, e = (step / NC) * 4 + el;
    const int within = e / (3 * V), r = e % (3 * V);
    g = r % 3;
    i = ((c / CP) * (H / P / V) + within * CP + c % CP) * V + r / 3;
  }
};

template <typename T, int H, int P>
constexpr size_t jm_rev_smem(int dim, int Lx) {
  return sizeof(T) * ((size_t)64 * RevOrder<T, H, P>::PITCH +
                      (dim == 2 ? mm_slot<T>(H) + (size_t)Lx * 64 * mm_tiles(H) * mm_lane_units(H) : 0));
}

template <typename T, int H, int DIM, int P>
__global__ __launch_bounds__(64 * mm_tiles(H), sizeof(T) == 8 && H == 64 ? 1 : 2) void k_jac_rev_mm(JmArgs<T> a) {
  using M = MM<T>;
  using acc_t = typename M::acc;
  using vec_t = typename M::vec;
  using R = RevOrder<T, H, P>;
  constexpr int NW = mm_tiles(H), NT = 64 * NW, KT = H / 4, V = M::V;
  constexpr int EU = mm_lane_units(H);   // units of a lane
  constexpr int KR = 3 * H / 4, PD = R::PITCH, PT = mm_pitch<T>(H);
  constexpr int NG = DIM == 2 ? 5 : 4;
  extern __shared__ __align__(16) unsigned char jsm[];
  T* D = reinterpret_cast<T*>(jsm);        // [4][16][PD] gate adjoints of a site
  T* X = D + 64 * PD;                      // 2D: [4][16][PT] adjoint of h'
  T* pend = X + mm_slot<T>(H);             // 2D: [Lx][NT][EU] from the row above, by column

  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int n = l & 15, q = l >> 4;
  const int j0 = mm_first<H>(w, q);
  const int N = a.N, Lx = a.Lx;
  const int ng = (a.ns + 15) / 16;
  const int seed = blockIdx.x / ng;
  const int sl0 = 16 * (blockIdx.x % ng) + n;
  const bool act = sl0 < a.ns;
  const int sl = min(sl0, a.ns - 1);
  const uint8_t* sg = a.sigma + (size_t)(a.s_base + sl) * N;
  const T* tp = a.tape + (size_t)sl * N * NG * H + j0;
  const T* hd = a.head + (size_t)sl * N * 4;
  T* ad = a.adj + ((size_t)seed * a.ns + sl) * N * NG * H + j0;

  // A operands: W_q^T rows (this wave's units), U1^T and U2^T rows
  const int jt = mm_unit<T, H>(w, n), ja = min(jt, H - 1);
  const bool arow = jt < H;
  T wr[KR], w1[DIM == 2 ? KT : 1], w2[DIM == 2 ? KT : 1];
#pragma unroll
  for (int t = 0; t < KR; ++t) {
    int g, i;
    R::input(t, q, g, i);
    const T x = a.w.bw[((size_t)(i / V) * H + ja) * 3 * V + g * V + i % V];
    wr[t] = arow ? x : (T)0;
  }
  if constexpr (DIM == 2) {
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const int i = 4 * t + q;
      const T* b = a.w.b2 + ((size_t)(i / V) * H + ja) * 2 * V + i % V;
      w1[t] = arow ? b[0] : (T)0;
      w2[t] = arow ? b[V] : (T)0;
    }
    for (int i = 0; i < Lx; ++i) {
      const T z[EU] = {};
      store4(pend + ((size_t)i * NT + tid) * EU, z);   // private to the thread
    }
  }
  // where this lane's 3 EU gate adjoints go
  int off[3][EU];
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int e = 0; e < EU; ++e) {
      int step, el;
      R::slot(g, j0 + e, step, el);
      off[g][e] = (el * 16 + n) * PD + step;
    }
  T U0[EU], U1[EU];
  load4(a.w.head + (2 * seed) * H + j0, U0);
  load4(a.w.head + (2 * seed + 1) * H + j0, U1);

  T carry[EU] = {};         // adjoint of h_{k} from site k + 1
  // the site's tape (1D: and h_{k-1}), requested a site ahead
  T t_[5][EU], hdn[4];
  int skn;
  auto fetch = [&](int k) {
#pragma unroll
    for (int g = 0; g < NG; ++g) load4(tp + ((size_t)k * NG + g) * H, t_[g]);
    if constexpr (DIM == 1) {
      if (k > 0) load4(a.states + ((size_t)(a.s_base + sl) * N + k - 1) * H + j0, t_[4]);
      else
#pragma unroll
        for (int e = 0; e < EU; ++e) t_[4][e] = (T)0;
    }
    load4(hd + 4 * k, hdn);
    skn = sg[k] & 1;
  };
  fetch(N - 1);
  for (int k = N - 1; k >= 0; --k) {
    T u[EU], r[EU], ag[EU], ht[EU], x[EU];
    const int sk = skn;
#pragma unroll
    for (int e = 0; e < EU; ++e) {
      u[e] = t_[0][e]; r[e] = t_[1][e]; ag[e] = t_[2][e]; ht[e] = t_[3][e]; x[e] = t_[4][e];
    }
    const T hc[4] = {hdn[0], hdn[1], hdn[2], hdn[3]};
    if (k > 0) fetch(k - 1);
    const int jr = DIM == 2 ? k / Lx : 0, kr = k - jr * Lx;
    const int col = (jr & 1) ? Lx - 1 - kr : kr;
    const bool hasV = DIM == 2 && jr > 0;
    T* pc = pend + ((size_t)col * NT + tid) * EU;
    T dz0, dz1;
    head_adjoint<T>(seed, sk, hc, dz0, dz1);
    T in[EU];
    if constexpr (DIM == 2) {
      load4(pc, in);
      // the neighbour along the path adds to it, unless k + 1 starts a row
      if (kr + 1 < Lx) {
#pragma unroll
        for (int e = 0; e < EU; ++e) in[e] += carry[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < EU; ++e) in[e] = carry[e];
    }
    T dpu[EU], dpr[EU], dg[EU], da[EU], dd[EU];
#pragma unroll
    for (int e = 0; e < EU; ++e) {
      T dh = dz0 * U0[e] + dz1 * U1[e];
      dh += in[e];
      const T dht = dh * u[e];
      const T du = dh * (ht[e] - x[e]);
      dd[e] = dh * ((T)1 - u[e]);
      da[e] = dht * ((T)1 - ht[e] * ht[e]);
      const T dr = da[e] * ag[e];
      dg[e] = da[e] * r[e];
      dpu[e] = du * u[e] * ((T)1 - u[e]);
      dpr[e] = dr * r[e] * ((T)1 - r[e]);
      D[off[0][e]] = dpu[e];
      D[off[1][e]] = dpr[e];
      D[off[2][e]] = dg[e];
    }
    T* ak = ad + (size_t)k * NG * H;
    if (act) {
      store4(ak, dpu); store4(ak + H, dpr); store4(ak + 2 * H, dg); store4(ak + 3 * H, da);
    }
    if (DIM == 1 && k == 0) break;         // nothing before the first site
    mm_sync<NW>();
    // adjoint of the cell input
    {
      acc_t c[R::NC];
      const T* p = D + (q * 16 + n) * PD;
#pragma unroll
      for (int i = 0; i < R::NC; ++i) c[i] = acc_t{(T)0, (T)0, (T)0, (T)0};
#pragma unroll
      for (int v = 0; v < KR / V; ++v) {
        const vec_t xv = *reinterpret_cast<const vec_t*>(p + V * v);
        const T* xs = reinterpret_cast<const T*>(&xv);
#pragma unroll
        for (int e = 0; e < V; ++e)
          c[(V * v + e) % R::NC] = M::mma(wr[V * v + e], xs[e], c[(V * v + e) % R::NC]);
      }
#pragma unroll
      for (int e = 0; e < EU; ++e)
#pragma unroll
        for (int pt = 0; pt < P; ++pt)
          if constexpr (R::CP == 2) dd[e] += c[2 * pt][e] + c[2 * pt + 1][e];
          else dd[e] += (c[4 * pt][e] + c[4 * pt + 1][e]) + (c[4 * pt + 2][e] + c[4 * pt + 3][e]);
    }
    if constexpr (DIM == 1) {
#pragma unroll
      for (int e = 0; e < EU; ++e) carry[e] = dd[e];
      mm_sync<NW>();                       // D is rewritten at the next site
    } else {
      if (act) store4(ak + 4 * H, dd);
      if (k == 0) break;                   // no predecessors
#pragma unroll
      for (int e = 0; e < EU; ++e) X[mm_place<T, H>(w, q, n, e)] = dd[e];
      mm_sync<NW>();
      // adjoints of the predecessors, a chain per part of the rows
      acc_t ch[P], cv[P];
      const T* p = X + (q * 16 + n) * PT;
#pragma unroll
      for (int pt = 0; pt < P; ++pt) ch[pt] = cv[pt] = acc_t{(T)0, (T)0, (T)0, (T)0};
#pragma unroll
      for (int v = 0; v < KT / V; ++v) {
        const vec_t xv = *reinterpret_cast<const vec_t*>(p + V * v);
        const T* xs = reinterpret_cast<const T*>(&xv);
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const int t = V * v + e, pt = t / (KT / P);
          ch[pt] = M::mma(w1[t], xs[e], ch[pt]);
          cv[pt] = M::mma(w2[t], xs[e], cv[pt]);
        }
      }
      T v4[EU];
#pragma unroll
      for (int e = 0; e < EU; ++e) {
        T sh = ch[0][e], sv = cv[0][e];
#pragma unroll
        for (int pt = 1; pt < P; ++pt) { sh += ch[pt][e]; sv += cv[pt][e]; }
        carry[e] = sh;
        v4[e] = hasV ? sv : (T)0;
      }
      // the column's slot now holds what the site below it receives
      store4(pc, v4);
    }
  }
}

// ------------------------------------------------------------ row assembly
// FP32: 32 x 32 x 2 products, FP64: 16 x 16 x 4 (lane l: A[l % TB][l / TB],
// B[l / TB][l % TB])
template <typename T> struct RowMM;
template <> struct RowMM<float> {
  typedef __attribute__((ext_vector_type(16))) float acc;
  static constexpr int TB = 32, E = 16;
  __device__ static acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int e, int kl) { return 8 * (e / 4) + 4 * kl + e % 4; }
};
template <> struct RowMM<double> {
  typedef f64x4r acc;
  static constexpr int TB = 16, E = 4;
  __device__ static acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int e, int kl) { return kl + 4 * e; }
};

template <typename T, int H, int DIM>
__global__ __launch_bounds__(256, 2) void k_jac_rows_mm(JmArgs<T> a) {
  using M = RowMM<T>;
  using acc_t = typename M::acc;
  constexpr int TB = M::TB, KS = 64 / TB;              // sites per K-step
  constexpr int WT = H / TB >= 4 ? 2 : 1;              // tiles per side of a wave's block
  constexpr int NB = H < TB ? 1 : H / (TB * WT);       // blocks per side
  constexpr int NM = DIM == 2 ? 5 : 3, NG = DIM == 2 ? 5 : 4;
  constexpr int ds = DIM == 1 ? 2 : 4;
  constexpr bool PAD = H < TB;                         // a tile wider than the model
  constexpr int UB = PAD ? 3 : 8;                      // K-steps requested together (d_h = 8, 36
                                                       // sites, 2048 rows: 8 47 us, 5 41.5, 3 40.6)
  extern __shared__ __align__(16) unsigned char rsm[];
  T* dz = reinterpret_cast<T*>(rsm);                   // [N][2] head adjoints
  int16_t* pre = reinterpret_cast<int16_t*>(dz + 2 * a.N);   // [3][N] the site, its predecessors, -1: none
  uint8_t* cod = reinterpret_cast<uint8_t*>(pre + 3 * a.N);  // [2][N] their spins, 2: none
  const int N = a.N, Lx = a.Lx;
  const int seed = blockIdx.x / a.ns, sl = blockIdx.x % a.ns;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kl = lane / TB, cl = lane % TB;
  const int cm = PAD ? min(cl, H - 1) : cl;            // further rows and columns are not stored
  const size_t s = (size_t)a.s_base + sl;
  const Layout& L = a.L;
  const T sc = a.scale;
  T* o = a.O + ((size_t)seed * a.Ns + s) * L.Np;
  const T* ad = a.adj + ((size_t)seed * a.ns + sl) * N * NG * H;
  const T* tp = a.tape + (size_t)sl * N * NG * H;
  const T* st = a.states + s * N * H;

  for (int k = tid; k < N; k += 256) {
    T h[4], d0, d1;
    load4(a.head + ((size_t)sl * N + k) * 4, h);
    const uint8_t* sg = a.sigma + s * N;
    head_adjoint<T>(seed, sg[k] & 1, h, d0, d1);
    dz[2 * k] = d0; dz[2 * k + 1] = d1;
    const int jr = DIM == 2 ? k / Lx : 0;
    const int p0 = k - jr * Lx > 0 ? k - 1 : -1, p1 = jr > 0 ? 2 * jr * Lx - 1 - k : -1;
    pre[k] = (int16_t)k; pre[N + k] = (int16_t)p0; pre[2 * N + k] = (int16_t)p1;
    cod[k] = p0 >= 0 ? sg[p0] & 1 : 2;
    cod[N + k] = p1 >= 0 ? sg[p1] & 1 : 2;
  }
  __syncthreads();

  // ---- weight blocks: matrix m is the sum over sites, last to first, of
  // adjoint x input; blocks of WT x WT tiles dealt to the four waves.  Bound
  // by the products (64 cycles each, four per two sites at d_h = 128): the
  // sites' predecessors come from a table, missing operands are masked on the
  // adjoint alone, and the next eight steps' operands are requested before the
  // current ones' products.
  for (int task = w; task < NM * NB * NB; task += 4) {
    const int m = task / (NB * NB), jb = (task / NB) % NB, cb = task % NB;
    const T* pa = ad + (m < 3 ? m : 4) * H + jb * TB * WT;
    // the input of site k: the cell input h' (2D), or a predecessor's state
    const bool own = DIM == 2 && m < 3;
    const T* pb = (own ? tp + 4 * H : st) + cb * TB * WT;
    const unsigned ldb = own ? NG * H : H;
    const int16_t* pm = pre + (own ? 0 : m == 4 ? 2 * N : N);
    acc_t acc[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int c = 0; c < WT; ++c)
#pragma unroll
        for (int e = 0; e < M::E; ++e) acc[i][c][e] = (T)0;
    auto load = [&](int u0, T (&x)[UB][WT], T (&y)[UB][WT]) {
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int k = N - 1 - (KS * (u0 + u) + kl), kc = max(k, 0);
        const int p = pm[kc];
        const bool on = k >= 0 && p >= 0;
        const unsigned oa = (unsigned)(kc * (NG * H) + cm), ob = (unsigned)max(p, 0) * ldb + cm;
#pragma unroll
        for (int i = 0; i < WT; ++i) {
          const T xa = pa[oa + i * TB];
          x[u][i] = on ? xa : (T)0;
          y[u][i] = pb[ob + i * TB];
        }
      }
    };
    auto products = [&](const T (&x)[UB][WT], const T (&y)[UB][WT]) {
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
          for (int c = 0; c < WT; ++c) acc[i][c] = M::mma(x[u][i], y[u][c], acc[i][c]);
    };
    const int nu = (N + KS - 1) / KS;                  // steps beyond it add zeros
    T a0[UB][WT], b0[UB][WT], a1[UB][WT], b1[UB][WT];
    load(0, a0, b0);
    for (int u0 = 0; u0 < nu; u0 += 2 * UB) {
      const bool more = u0 + UB < nu;
      if (more) load(u0 + UB, a1, b1);
      products(a0, b0);
      if (!more) break;
      if (u0 + 2 * UB < nu) load(u0 + 2 * UB, a0, b0);
      products(a1, b1);
    }
    const size_t off = m == 0 ? L.Wu : m == 1 ? L.Wr : m == 2 ? L.Wh : m == 3 ? L.U1 : L.U2;
    const unsigned ldq = m < 2 ? H + ds : H;
    T* om = o + off + cb * TB * WT;
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int e = 0; e < M::E; ++e) {
        const unsigned at = ((jb * WT + i) * TB + M::row(e, kl)) * ldq + cl;
#pragma unroll
        for (int c = 0; c < WT; ++c)
          if (!PAD || (M::row(e, kl) < H && cl < H)) om[at + c * TB] = acc[i][c][e] * sc;
      }
  }

  // ---- biases, one-hot input columns and the head: thread j sums its unit
  // over the sites, last to first; job 0: u, 1: r, 2: candidate, 3: head
  constexpr int JS = H < 64 ? 64 : H, NJ = 256 / JS;   // d_h <= 64: a wave per job
  const int j = tid % JS;
  for (int job = tid / JS; job < 4 && j < H; job += NJ) {
    T b = (T)0, b2 = (T)0, gx[ds];
#pragma unroll
    for (int c = 0; c < ds; ++c) gx[c] = (T)0;
    const T* p1 = job < 3 ? ad + job * H + j : st + j;   // job 2: b_h from row 2, the rest from 3
    const T* p2 = ad + (job == 2 ? 3 : job & 1) * H + j;
    const unsigned ld1 = job < 3 ? NG * H : H;
    for (int k1 = N - 1; k1 >= 0; k1 -= 8) {
      T v[8], x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const unsigned k = (unsigned)max(k1 - i, 0);
        v[i] = p1[k * ld1];
        x[i] = p2[k * (unsigned)(NG * H)];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bool on = k1 - i >= 0;
        const int k = max(k1 - i, 0);
        const T vi = on ? v[i] : (T)0, xi = on ? x[i] : (T)0;
        const T d0 = job == 3 ? dz[2 * k] * vi : vi, d1 = job == 3 ? dz[2 * k + 1] * vi : xi;
        b += d0;
        b2 += d1;
        const int c0 = cod[k];
        gx[0] += c0 == 0 ? xi : (T)0;
        gx[1] += c0 == 1 ? xi : (T)0;
        if constexpr (DIM == 2) {
          const int c1 = cod[N + k];
          gx[2] += c1 == 0 ? xi : (T)0;
          gx[3] += c1 == 1 ? xi : (T)0;
        }
      }
    }
    if (job < 2) {
      const size_t off = job == 0 ? L.Wu : L.Wr;
#pragma unroll
      for (int c = 0; c < ds; ++c) o[off + (size_t)j * (H + ds) + H + c] = gx[c] * sc;
      o[(job == 0 ? L.bu : L.br) + j] = b * sc;
    } else if (job == 2) {
#pragma unroll
      for (int c = 0; c < ds; ++c) o[L.Win + (size_t)j * ds + c] = gx[c] * sc;
      o[L.bh + j] = b * sc;
      o[L.bin + j] = b2 * sc;
    } else {
      const size_t hU = seed == 0 ? L.U : L.Uphi, zU = seed == 0 ? L.Uphi : L.U;
      o[hU + j] = b * sc; o[hU + H + j] = b2 * sc;
      if (a.cplx) { o[zU + j] = (T)0; o[zU + H + j] = (T)0; }
      if (j < 2) {
        T g = (T)0;
        for (int k = N - 1; k >= 0; --k) g += dz[2 * k + j];
        o[(seed == 0 ? L.c : L.cphi) + j] = g * sc;
        if (a.cplx) o[(seed == 0 ? L.cphi : L.c) + j] = (T)0;
      }
    }
  }
}

// ---- launch of one chunk

template <typename T, int H, int DIM, int P>
static int jm_chunk(const JmArgs<T>& a, hipStream_t s) {
  static std::once_flag once;   // more than 64 KiB of dynamic shared memory
  hipError_t attr = hipSuccess;
  std::call_once(once, [&] {
    attr = hipFuncSetAttribute((const void*)k_jac_rev_mm<T, H, DIM, P>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)MM_LDS);
  });
  MINSR_HIP(attr);
  const unsigned seeds = a.cplx ? 2 : 1;
  const long long pairs = (long long)a.ns * a.N;
  if (pairs > 65536) k_jac_head<T, H, 64><<<(unsigned)((pairs + 255) / 256), 256, 0, s>>>(a);
  else k_jac_head<T, H, 16><<<(unsigned)((pairs + 63) / 64), 256, 0, s>>>(a);
  MINSR_CHECK_LAUNCH();
  k_jac_rev_mm<T, H, DIM, P><<<seeds * (unsigned)((a.ns + 15) / 16), 64 * mm_tiles(H),
                            jm_rev_smem<T, H, P>(DIM, a.Lx), s>>>(a);
  MINSR_CHECK_LAUNCH();
  k_jac_rows_mm<T, H, DIM><<<seeds * (unsigned)a.ns, 256, a.N * (2 * sizeof(T) + 8), s>>>(a);
  MINSR_CHECK_LAUNCH();
  return MINSR_OK;
}

// values per sample and site of the tape, the head and the adjoints
inline size_t jm_site_elems(int dim, int H, int cplx) {
  return (size_t)(dim == 2 ? 5 : 4) * H * (cplx ? 3 : 2) + 4;
}

// samples first to last in chunks of the tape; the forward pass's tape serves
// a call of one chunk, otherwise each chunk's is formed here
template <typename T, typename REC, typename RUN>
static int jm_run(minsr_model* m, JmArgs<T> a, bool have_tape, REC rec, RUN run, hipStream_t s) {
  a.tape = (const T*)m->gates; a.adj = (T*)m->jadj; a.head = (T*)m->jhead;
  for (int b = 0; b < a.Ns; b += m->gates_ns) {
    a.s_base = b;
    a.ns = a.Ns - b < m->gates_ns ? a.Ns - b : m->gates_ns;
    if (!have_tape) {
      RecCall c{};
      c.Ns = a.ns; c.sigma = const_cast<uint8_t*>(a.sigma) + (size_t)b * a.N;
      c.store_every = 1; c.gates = m->gates;
      if (const int rc = rec(m, 1, c, s)) return rc;
    }
    if (const int rc = run(a)) return rc;
  }
  return MINSR_OK;
}

template <typename T>
static JmArgs<T> jm_args(const minsr_model* m, const Work<T>& w, int Ns, const uint8_t* sigma,
                         const void* states, void* O) {
  JmArgs<T> a{};
  a.w = w; a.L = m->L;
  a.N = m->N; a.Lx = m->d.Lx; a.Ns = Ns; a.zero_mag = m->d.zero_mag; a.cplx = m->cplx;
  a.sigma = sigma; a.states = (const T*)states; a.O = (T*)O;
  a.scale = (T)(1.0 / std::sqrt((double)Ns));
  return a;
}

}  // namespace minsr
