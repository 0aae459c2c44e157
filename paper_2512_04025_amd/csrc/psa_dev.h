// Device-side helpers shared by the PSA kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace psa {

typedef uint16_t bf16_t;  // raw bfloat16 bits

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even; NaN stays NaN.  Two at a time: one conversion instruction.
typedef __attribute__((ext_vector_type(2))) float f32x2;
__device__ __forceinline__ uint32_t f32_to_bf16_pair(float x, float y) {   // x in the low half
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x, y}), bf16x2));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)f32_to_bf16_pair(f, f); }

// Element-type traits: a 16-byte vector of VEC elements, widened to float and narrowed back.
template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int VEC = 4;
  __device__ static __forceinline__ void load(const float* p, float* out) { widen(*reinterpret_cast<const u32x4*>(p), out); }
  __device__ static __forceinline__ void widen(u32x4 x, float* out) {
    f32x4 v = __builtin_bit_cast(f32x4, x);
    out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
  }
  __device__ static __forceinline__ u32x4 pack(const float* in) { return __builtin_bit_cast(u32x4, (f32x4{in[0], in[1], in[2], in[3]})); }
  __device__ static __forceinline__ void store(float* p, const float* in) { *reinterpret_cast<u32x4*>(p) = pack(in); }
  __device__ static __forceinline__ float to_f32(float x) { return x; }
  __device__ static __forceinline__ float from_f32(float x) { return x; }
};
template <> struct Elem<bf16_t> {
  static constexpr int VEC = 8;
  __device__ static __forceinline__ void load(const bf16_t* p, float* out) { widen(*reinterpret_cast<const u32x4*>(p), out); }
  __device__ static __forceinline__ void widen(u32x4 v, float* out) {
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = __uint_as_float(w[i] << 16);
      out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  __device__ static __forceinline__ u32x4 pack(const float* in) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = f32_to_bf16_pair(in[2 * i], in[2 * i + 1]);
    return u32x4{w[0], w[1], w[2], w[3]};
  }
  __device__ static __forceinline__ void store(bf16_t* p, const float* in) { *reinterpret_cast<u32x4*>(p) = pack(in); }
  __device__ static __forceinline__ float to_f32(bf16_t x) { return bf16_to_f32(x); }
  __device__ static __forceinline__ bf16_t from_f32(float x) { return f32_to_bf16(x); }
};

// Four consecutive elements for the fp32-arithmetic kernels.  The caller's tensors need no more than element
// alignment there (the memory pipeline takes 16-byte accesses at any address), so the vector types do not
// claim more.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t u16x4_any __attribute__((ext_vector_type(4), aligned(2)));
template <typename T> struct Four;
template <> struct Four<float> {
  typedef f32x4 raw;
  __device__ static __forceinline__ raw load(const float* p) { return *reinterpret_cast<const f32x4_any*>(p); }
  __device__ static __forceinline__ f32x4 widen(raw r) { return r; }
  __device__ static __forceinline__ void store(float* p, f32x4 x) { *reinterpret_cast<f32x4_any*>(p) = x; }
};
template <> struct Four<bf16_t> {
  typedef uint16_t raw __attribute__((ext_vector_type(4)));
  __device__ static __forceinline__ raw load(const bf16_t* p) { return *reinterpret_cast<const u16x4_any*>(p); }
  __device__ static __forceinline__ f32x4 widen(raw r) {
    return f32x4{bf16_to_f32(r[0]), bf16_to_f32(r[1]), bf16_to_f32(r[2]), bf16_to_f32(r[3])};
  }
  __device__ static __forceinline__ void store(bf16_t* p, f32x4 x) {
    *reinterpret_cast<u16x4_any*>(p) = __builtin_bit_cast(u16x4_any, (u32x2{f32_to_bf16_pair(x[0], x[1]), f32_to_bf16_pair(x[2], x[3])}));
  }
};

__device__ __forceinline__ bool not_finite(f32x4 x) {
  bool bad = false;
#pragma unroll
  for (int u = 0; u < 4; ++u) bad |= (__float_as_uint(x[u]) & 0x7f800000u) == 0x7f800000u;
  return bad;
}

// f(integral_constant 0), f(1) .. f(N - 1)
template <int N, int I = 0, typename F> __device__ __forceinline__ void each(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    each<N, I + 1>(f);
  }
}

// x ^ a constant, made where it is used: an address per constant would otherwise be held in a register over the whole loop
template <int C> __device__ __forceinline__ uint32_t flip(uint32_t x) {
  if (C == 0) return x;
  uint32_t y;
  asm volatile("v_xor_b32 %0, %1, %2" : "=v"(y) : "n"(C), "v"(x));
  return y;
}

// the lane's number, made where it is used: what depends on it is worked out again instead of held over the stage loop
__device__ __forceinline__ int lane_again() {
  int x;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
  return x;
}

// Place of a bfloat16 row's 16-byte chunks in LDS for operands of 32 rows (two lanes a row): chunk ^ row_swizzle32(row).  16 consecutive
// rows are at 16 different places, and the four rows of a transposing group in four different 64-byte groups.
template <int D> __host__ __device__ constexpr int row_swizzle32(int row) {
  return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

// float32 on the bfloat16 matrix cores: x = h + m + l exactly, three bfloat16 (8 bits each, the remainders rounded to nearest and signed), so that
// a product is the six terms down to 2^-16 of it (h h, h m, m h, m m, h l, l h); the three that are left out are of the order of 2^-25 of it.
// Not for values that are not finite (or round to infinity): their m and l are NaN.  Nor for those whose last bits lie below 2^-133, the smallest
// bfloat16 (of 24 bits: values below 2^-110).
struct Split2 { uint32_t h, m, l; };                 // of two neighbours: the first in the low halves
__device__ __forceinline__ Split2 split2(float a, float b) {
  Split2 s;
  s.h = f32_to_bf16_pair(a, b);
  a -= __uint_as_float(s.h << 16);
  b -= __uint_as_float(s.h & 0xffff0000u);
  s.m = f32_to_bf16_pair(a, b);
  a -= __uint_as_float(s.m << 16);
  b -= __uint_as_float(s.m & 0xffff0000u);
  s.l = f32_to_bf16_pair(a, b);
  return s;
}

// Of bfloat16 pairs: whether one is large or not finite; whether one is small, but not 0, so that a float32 value rounded to it may not be the sum
// of its planes.  (Plain code: in assembly, an instruction less, it was not moved between the products, 6000 tokens at d = 64 231 -> 249 us.)
typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;
struct PairRange {
  u16x2 least = {0xffff, 0xffff}, most = {0, 0};
  __device__ __forceinline__ void add(uint32_t pair) {
    const u16x2 size = __builtin_bit_cast(u16x2, pair) << (uint16_t)1;
    least = __builtin_elementwise_min(least, (u16x2)(size - (uint16_t)1));   // (0 is the largest)
    most = __builtin_elementwise_max(most, size);
  }
  __device__ __forceinline__ bool small() const { return (least[0] < least[1] ? least[0] : least[1]) < 0x11ff; }   // below 2^-109
  __device__ __forceinline__ bool large() const { return (most[0] > most[1] ? most[0] : most[1]) >= 0xcf00; }      // 2^80
};

__device__ __forceinline__ int ilog2(int x) { return 31 - __clz(x); }

// A row of the level map -> its kept blocks grouped by level (ascending inside a level) and the number per level, in LDS, by
// the NW wavefronts of a workgroup (which then wait for each other).  Rows of at most ROW_LISTS_NK blocks.
constexpr int ROW_LISTS_NK = 128;
template <int NW>
__device__ __forceinline__ void row_lists(const uint8_t* __restrict__ m, int nk, int H, uint16_t* list, int* cnt, int wave, int lane) {
  int lv[ROW_LISTS_NK / 64];
#pragma unroll
  for (int c = 0; c < ROW_LISTS_NK / 64; ++c) lv[c] = c * 64 + lane < nk ? (int)m[c * 64 + lane] : 0;
  const uint64_t below = (1ull << lane) - 1ull;
  int first = 0;
  for (int h = 1; h <= H; ++h) {
    int before[ROW_LISTS_NK / 64], n = 0;
#pragma unroll
    for (int c = 0; c < ROW_LISTS_NK / 64; ++c) {
      const uint64_t mask = __ballot(lv[c] == h);
      before[c] = n + __popcll(mask & below);
      n += __popcll(mask);
    }
    if (NW == 1 || h % NW == wave) {
#pragma unroll
      for (int c = 0; c < ROW_LISTS_NK / 64; ++c)
        if (lv[c] == h) list[first + before[c]] = (uint16_t)(c * 64 + lane);
      if (lane == 0) cnt[h - 1] = n;
    }
    first += n;
  }
}

// Causal work on the 8 XCDs, whose rows (or columns) differ in length by up to the whole sequence: every XCD takes as many whole heads as
// all can have, one after the other, and of the heads that are left every eighth item.  (Contiguous runs gave one XCD the long half
// of a shared head and its neighbour the short one.)
__host__ __device__ inline int xcd_slots(int heads, int per_head) { return heads / 8 * per_head + (heads % 8 * per_head + 7) / 8; }
__device__ __forceinline__ bool xcd_item(int heads, int per_head, int xcd, int slot, int& head, int& item) {
  const int each = heads / 8, rest = heads % 8;
  if (slot < each * per_head) {
    head = xcd * each + slot / per_head;
    item = slot % per_head;
    return true;
  }
  const int k = (slot - each * per_head) * 8 + xcd;
  if (k >= rest * per_head) return false;
  head = each * 8 + k % rest;
  item = k / rest;
  return true;
}
// ... and where an item is
__device__ __forceinline__ void xcd_of_item(int heads, int per_head, int head, int item, int& xcd, int& slot) {
  const int each = heads / 8, rest = heads % 8;
  if (head < each * 8) {
    xcd = head / each;
    slot = head % each * per_head + item;
  } else {
    const int k = item * rest + head - each * 8;
    xcd = k & 7;
    slot = each * per_head + (k >> 3);
  }
}

}  // namespace psa
