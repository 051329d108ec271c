// The 16 x 16 x 4 FP32 and FP64 matrix products as the recurrence and its
// reverse pass use them, and the shared-memory layout of their operands.
#pragma once

#include "mfma16.hpp"
#include "model.hpp"

namespace minsr {

typedef __attribute__((ext_vector_type(4))) float f32x4r;
typedef __attribute__((ext_vector_type(4))) double f64x4r;

// Tiles of 16 units of a hidden width, and the units of a lane in a tile's
// result: four, or two at d_h = 8, where the eight rows that are left have
// zero weights and land in result elements that nothing reads.
__host__ __device__ constexpr int mm_tiles(int H) { return (H + 15) / 16; }
__host__ __device__ constexpr int mm_lane_units(int H) { return H < 16 ? 2 : 4; }

// Lane l of a product: A[l % 16][l / 16], B[l / 16][l % 16]; result element v
// is unit 4 (l / 16) + v of the tile, column l % 16 (the FP64 result rows are
// permuted to that by the order of the A rows).  Both instructions add their
// four products in ascending k as a chain of fused multiply-adds (compared
// with such chains over 5e4 random tiles each: all bits equal).
template <typename T> struct MM;
template <> struct MM<float> {
  typedef f32x4r acc;
  typedef float4 vec;                 // one shared-memory read
  static constexpr int V = 4;         // its elements; also the weight packing's vector
  __device__ static int row(int r) { return r; }   // unit of A row r
  __device__ static acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <> struct MM<double> {
  typedef f64x4r acc;
  typedef double2 vec;
  static constexpr int V = 2;
  // result row r lies in lane group r % 4, element r / 4
  __device__ static int row(int r) { return 4 * (r & 3) + (r >> 2); }
  __device__ static acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// a lane's consecutive units as one (FP64: two, d_h = 8 one) 16-byte accesses
__device__ inline void load4(const float* p, float (&v)[4]) {
  const float4 x = *reinterpret_cast<const float4*>(p);
  v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
}
__device__ inline void load4(const double* p, double (&v)[4]) {
  const double2 x = *reinterpret_cast<const double2*>(p), y = *reinterpret_cast<const double2*>(p + 2);
  v[0] = x.x; v[1] = x.y; v[2] = y.x; v[3] = y.y;
}
__device__ inline void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline void store4(double* p, const double (&v)[4]) {
  *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
  *reinterpret_cast<double2*>(p + 2) = make_double2(v[2], v[3]);
}

__device__ inline void load4(const double* p, double (&v)[2]) {
  const double2 x = *reinterpret_cast<const double2*>(p);
  v[0] = x.x; v[1] = x.y;
}
__device__ inline void store4(double* p, const double (&v)[2]) {
  *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
}

// sums over lanes 16 and 32 apart, by lane swaps
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
// value of the lane that DPP control C names (within rows of 16 lanes)
template <int C> __device__ inline float row_lane(float v) { return mf16::dpp_f<C>(v); }
template <int C> __device__ inline double row_lane(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, C, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), C, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}
// sum over groups of W lanes in every lane, in the order of an xor butterfly
// from W / 2 down (W = 8: up), on the VALU: a row's values repeat with the
// distances already added, so a rotation reaches the partner's value
template <int W, typename T> __device__ inline T unit_sum(T v) {
  if constexpr (W == 64) v = xor32_sum(v);
  if constexpr (W >= 32) v = xor16_sum(v);
  if constexpr (W >= 16) {
    v += row_lane<0x128>(v);                // rotated by 8
    v += row_lane<0x124>(v);
    v += row_lane<0x122>(v);
    v += row_lane<0x121>(v);
  } else {
    v += row_lane<0xB1>(v);                 // quad_perm [1, 0, 3, 2]
    v += row_lane<0x4E>(v);                 // quad_perm [2, 3, 0, 1]
    v += row_lane<0x141>(v);                // row_half_mirror
  }
  return v;
}
// value of lane L (the same in every lane)
template <int L> __device__ inline float wave_lane(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), L));
}
template <int L> __device__ inline double wave_lane(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, L);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), L);
  return __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}

// workgroup barrier ordering shared memory only; a single wave needs a fence
template <int NW> __device__ inline void mm_sync() {
  if constexpr (NW == 1) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    mf16::lds_barrier();
  }
}

// A state (or adjoint) vector of 16 sequences as a B operand in shared
// memory: [unit % 4][sequence][unit / 4], rows padded so that the 16-byte
// reads of a quarter wave and the writes fall on different banks
template <typename T> constexpr int mm_pitch(int H) { return H / 4 + MM<T>::V; }
template <typename T> constexpr size_t mm_slot(int H) { return (size_t)64 * mm_pitch<T>(H); }
// first unit of a lane (wave w, lane group q); unit of A row r of a wave's
// tile, H or above: none; place of a lane's unit e in such a vector
template <int H> __device__ inline int mm_first(int w, int q) { return H < 16 ? 2 * q : 16 * w + 4 * q; }
template <typename T, int H> __device__ inline int mm_unit(int w, int r) {
  return H < 16 ? 2 * (r & 3) + (r >> 2) + (r >> 3) * H : 16 * w + MM<T>::row(r);
}
template <typename T, int H> __device__ inline int mm_place(int w, int q, int n, int e) {
  return H < 16 ? ((2 * (q & 1) + e) * 16 + n) * mm_pitch<T>(H) + (q >> 1)
                : (e * 16 + n) * mm_pitch<T>(H) + 4 * w + q;
}

constexpr size_t MM_LDS = 160 * 1024;

}  // namespace minsr
