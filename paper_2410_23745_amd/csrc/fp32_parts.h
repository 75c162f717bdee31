// fp32 values as sums of three bf16 parts, for fp32 contractions on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 values (8 significant bits each): x = h + m + l with h = bf16(x),
// m = bf16(x - h), l = x - h - m.  A product of two fp32 values is then nine bf16 products, each exact in fp32, of which
// the three smallest (m*l, l*m, l*l) are left out; the six others are accumulated in fp32 by
// v_mfma_f32_16x16x32_bf16.  Six of them take 96 cycles for 32 terms where v_mfma_f32_16x16x4_f32 takes 256.
// What is left out is together below 0.996 * 2^-24 of the product (every pair of mantissas' largest m and l; 0.09 * 2^-24
// in the mean square), about one more rounding of it: a result with a single term that is not zero can be 2 * 2^-24 off where
// the fp32 instructions give 2^-24, and sums are closer than theirs, because the large sum is rounded less often.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace syno {
namespace {

constexpr int kPlanes = 3;

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t round_pair(float lo, float hi) {      // v_cvt_pk_bf16_f32: to nearest even
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// (x0, x1) -> the two values' parts, packed pairwise, times 2^24: the bf16 matrix instructions take subnormal operands for
// zero, and a multiple of 2^-149 becomes one of 2^-125, so that no part of any fp32 value, subnormal ones included, is a
// subnormal; what the instructions drop of a sum is below 2^-126 / 2^48.  The last
// remainder has at most 8 significant bits: its upper half is the value itself.  An infinity, a NaN or a value above 2^104
// leaves a NaN in m or l, so every result that it takes part in is a NaN and is summed again when it is stored; so
// are sums beyond 2^80.
constexpr float kPartScale = 16777216.f, kResultScale = 1.f / (16777216.f * 16777216.f);
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  x0 *= kPartScale;
  x1 *= kPartScale;
  h = round_pair(x0, x1);
  const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
  m = round_pair(r0, r1);
  const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xffff0000u);
  l = __builtin_amdgcn_perm(__float_as_uint(s1), __float_as_uint(s0), 0x07060302u);
}

// Whether a result is what the parts' sum is
constexpr float kMostResult = 3.4028234663852886e38f;
__device__ __forceinline__ bool trusted_result(float v) { return fabsf(v) <= kMostResult; }

}  // namespace
}  // namespace syno
