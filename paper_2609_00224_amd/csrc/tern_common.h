// Pieces shared by the FP4 matrix-core kernels (tern_mfma.hip, tern_solo.hip):
// the decode table, the digit split of the activations, the instruction.
// Internal to the library.
#ifndef QTEA_TERN_COMMON_H_
#define QTEA_TERN_COMMON_H_

#include "grouped_plan.h"

namespace qtea_grouped {

constexpr int kDigits = 6;
constexpr uint32_t kDigitBias = 0x21084210u;  // 16 * (1 + 32 + ... + 32^5)
constexpr int kUnitMfma = 4;                  // instructions per 16-row tile, unit and result block
// Decode table rows of 256 bytes: 32 copies of the entry, and 128 bytes that
// hold the small per-wave and per-workgroup areas ("holes").  The debug
// build (QTEA_DEBUG) keeps the rows of the unused byte values 243..255 (zero
// entries) so that such a byte, which it reports as NaN, reads its own row.
#ifdef QTEA_DEBUG
constexpr int kTabRows = 256;
#else
constexpr int kTabRows = kCodes;
#endif
constexpr int kTab = kTabRows * 256;
constexpr int kHoleBytes = kCodes * 128;
// Staging area of a wave and tile: 32 columns' residual values of the tile (1 KiB)
// and their position words; the part end transposes its sums through it.
constexpr int kStage = 1024 + 128;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) f32x4u gf32x4u;
typedef __attribute__((address_space(1))) const u32x2 gu32x2;
template <class T>
using lds_t = __attribute__((address_space(3))) T;

template <class T>
__device__ __forceinline__ T lds_read(uint32_t a) {
  return *(const lds_t<T>*)(size_t(a));
}
template <class T>
__device__ __forceinline__ void lds_write(uint32_t a, T v) {
  *(lds_t<T>*)(size_t(a)) = v;
}

// Address of byte o of the space formed by the unused halves of the table rows.
__device__ __forceinline__ constexpr uint32_t hole(uint32_t o) { return o + (o & ~127u) + 128u; }

__device__ __forceinline__ half8 as_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const u32x4 v = {a, b, c, d};
  return __builtin_bit_cast(half8, v);
}

// The five codes of byte value c as FP4 nibbles (digit 0 lowest).
__device__ __forceinline__ uint32_t tern_entry(uint32_t c) {
  uint32_t e = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const uint32_t r = c / 3, d = c - 3 * r;
    e |= (d == 0 ? 0xAu : (d == 1 ? 0u : 0x2u)) << (4 * i);
    c = r;
  }
  return e;
}

// One instruction: digits (FP6) x codes (FP4) with the digits' block scales
// in byte I of sc.
template <int I>
__device__ __forceinline__ f32x4 tern_mfma(const u32x4 a, const u32x2 a2, const uint32_t (&e)[4], const f32x4 c,
                                           const uint32_t sc) {
  const i32x8 A = {int(a.x), int(a.y), int(a.z), int(a.w), int(a2.x), int(a2.y), 0, 0};
  const i32x8 B = {int(e[0]), int(e[1]), int(e[2]), int(e[3]), 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, B, c, 2, 4, I, int(sc), 0, 0x7f7f7f7f);
}

// Max over the four lanes of a quad.
__device__ __forceinline__ uint32_t quad_max(uint32_t x) {
  const uint32_t y = max(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xB1, 0xf, 0xf, true)));   // 1,0,3,2
  return max(y, uint32_t(__builtin_amdgcn_update_dpp(0, int(y), 0x4E, 0xf, 0xf, true)));               // 2,3,0,1
}

// The lane index, opaque: what is derived from it is computed where it is
// used instead of being held in registers across the unit loop.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// The products a_i = v_i x_i of one pack's five columns (v and x in the
// low halves of v5 and x5): exact, 22 bits each.
__device__ __forceinline__ void tern_products(const uint32_t (&v5)[5], const uint32_t (&x5)[5], float (&a)[5]) {
#pragma unroll
  for (int i = 0; i < 5; ++i)
    a[i] = float(__builtin_bit_cast(_Float16, uint16_t(v5[i] & 0xffffu))) * float(__builtin_bit_cast(_Float16, uint16_t(x5[i])));
}

// The sum over the four lanes of a quad.
__device__ __forceinline__ uint32_t quad_sum(uint32_t x) {
  const uint32_t y = x + uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xB1, 0xf, 0xf, true));    // 1,0,3,2
  return y + uint32_t(__builtin_amdgcn_update_dpp(0, int(y), 0x4E, 0xf, 0xf, true));                // 2,3,0,1
}

// The fixed point of one pack's five a_i and of the other three packs of its
// quad (a block of 20 columns): f[i] = a_i 2^(154 - ex) rounded to a whole
// number, |f| <= 2^28; ex the block's biased exponent, mx its largest |a| as bits.
__device__ __forceinline__ float tern_unit(uint32_t ex) { return __builtin_bit_cast(float, (281u - ex) << 23); }
__device__ __forceinline__ void tern_fixed(const float (&a)[5], float (&f)[5], uint32_t& ex, uint32_t& mx) {
  mx = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) mx = max(mx, __builtin_bit_cast(uint32_t, a[i]) & 0x7fffffffu);
  mx = quad_max(mx);
  ex = max(mx >> 23, 64u);  // |a| >= 2^-48 unless zero
#pragma unroll
  for (int i = 0; i < 5; ++i) f[i] = __builtin_rintf(a[i] * tern_unit(ex));
}

// Whether the wave's slice needs a second set of ND digits, for what the first
// leaves of the a_i: then f becomes that, in units of 2^(1 - 5 ND) of the first's.
// The first set rounds an a_i below 2^-6 of its block's power of two to 2^-28 of
// it: nothing beside the block's other columns, unless many of them are that
// small.  Then a row whose codes at the few large columns are 0 would be left
// with the rounding (an outlier of 16000 among N(0, 1): 2.5e-6 of such a row at
// K = 4096, with the second set 8e-8; fp32 sums: 1.1e-7).  The line is five of
// the block's columns, in a block that has a whole pack below about 2^-3 (its
// top digits `top` are 0: a test that costs the other slices two
// instructions, where the count below cost 0.15 to 0.3 us per unit).  N(0, 1)
// activations pass the line in one of 500 slices.
template <int ND>
__device__ __forceinline__ bool tern_rest(const float (&a)[5], float (&f)[5], uint32_t ex, uint32_t top) {
  if (__builtin_expect(__ballot(top == 0u) == 0, 1)) return false;
  uint32_t low = 0;
  bool left = false;
  float r[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    r[i] = __builtin_fmaf(a[i], tern_unit(ex), -f[i]);  // (exact: fewer bits than a_i)
    left |= r[i] != 0.0f;
    low += __builtin_fabsf(f[i]) < 0x1p21f ? 1u : 0u;
  }
  low = quad_sum(low);
  if (__builtin_expect(__ballot(left && low >= 5u) == 0, 1)) return false;  // (zeros are small and leave nothing)
#pragma unroll
  for (int i = 0; i < 5; ++i) f[i] = __builtin_rintf(r[i] * float(1 << (5 * ND - 1)));
  return true;
}

// The base-32 digits of f: the five codes of digit l at bits 6 i of P[l].
template <int ND>
__device__ __forceinline__ void tern_digits(const float (&f)[5], uint32_t (&P)[ND]) {
  uint32_t uq[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) uq[i] = uint32_t(int(f[i])) + (kDigitBias & ((1u << (5 * ND)) - 1u));
#pragma unroll
  for (int l = 0; l < ND; ++l) {
    uint32_t F = 0;  // per column the digit + 16 at bits 6 i .. 6 i + 4
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const uint32_t sh = 6 * i >= 5 * l ? uq[i] << (6 * i - 5 * l) : uq[i] >> (5 * l - 6 * i);
      F |= sh & (31u << (6 * i));
    }
    // to sign (bit 6 i + 5) and magnitude 0..16
    constexpr uint32_t kOnes = 0x01041041u;
    const uint32_t s = ~(F >> 4) & kOnes;
    P[l] = ((F & (15u * kOnes)) ^ ((s << 4) - s)) + (s + (s << 5));
  }
}
// E8M0 scale of digit l of such a block, in the first set and in a second of
// ND (NaN when an activation is not finite).
__device__ __forceinline__ uint8_t tern_scale(uint32_t ex, uint32_t mx, int l) {
  return uint8_t(mx >= 0x7f800000u ? 255u : ex + 5u * uint32_t(l) - 24u);
}
template <int ND>
__device__ __forceinline__ uint8_t tern_rest_scale(uint32_t ex, uint32_t mx, int l) {
  return uint8_t(mx >= 0x7f800000u ? 255u : ex + 5u * uint32_t(l) - uint32_t(23 + 5 * ND));
}
// The value of the quad's lane 1 or 2, in its lane 0.
__device__ __forceinline__ uint32_t quad_next(uint32_t x) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xF9, 0xf, 0xf, true));
}
__device__ __forceinline__ uint32_t quad_next2(uint32_t x) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xFE, 0xf, 0xf, true));
}

}  // namespace qtea_grouped

#endif  // QTEA_TERN_COMMON_H_
