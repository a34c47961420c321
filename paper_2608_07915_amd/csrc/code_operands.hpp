// Packed codes as matrix-core operands, shared by the reconstruction and per-layer kernels.
#pragma once
#include "device_common.hpp"

namespace spectra_dev {

typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;

// ---------------------------------------------------------------------------
// Codes of one token as fp16 matrix operands: the B payload words w[0 .. B) hold 32 codes
// at width B (a group of 32, or half of a group of 64). Codes j and j + 16 lie B 16-bit
// halves apart at the same bit offset, so joining half i with half i + B puts
// them at the same offset of the two halves of one register, and one shift and one mask
// serve both; OR-ing in the exponent of 1024 and subtracting 1024 + 2^(B-1) (both
// exact) gives the two as fp16 integers centered on 0. About 1.6 instructions per code
// against 2.5 for single extraction and conversion. Element 2i + e of codes_f16(k) is code
// 4k + i + 16e: the other operand of a product is laid out to match.
// ---------------------------------------------------------------------------
template <int B>
__device__ __forceinline__ void join_halves(const uint32_t (&w)[8], uint32_t (&Z)[8]) {
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const uint32_t sel = ((i & 1) ? 0x0302u : 0x0100u) | (((i + B) & 1) ? 0x07060000u : 0x05040000u);
    Z[i] = __builtin_amdgcn_perm(w[(i + B) >> 1], w[i >> 1], sel);
  }
}
template <int B>
__device__ __forceinline__ f16x8 codes_f16(const uint32_t (&Z)[8], int k, uint32_t magic) {
  constexpr uint32_t M = (1u << B) - 1u, MM = M | (M << 16);
  const _Float16 off = (_Float16)(1024.0f + (float)(1 << (B - 1)));
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int bit = (4 * k + i) * B, z = bit >> 4, p = bit & 15;
    uint32_t v;
    if (p + B <= 16) {
      v = ((Z[z] >> p) & MM) | magic;
    } else {  // the code continues in the next pair of halves
      const int nlo = 16 - p;
      const uint32_t L = (1u << nlo) - 1u, H = M & ~L;
      v = ((Z[z] >> p) & (L | (L << 16))) | magic;
      v |= (Z[z + 1] << nlo) & (H | (H << 16));
    }
    r[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, v) - f16x2{off, off});
  }
  return __builtin_bit_cast(f16x8, r);
}
// The exponent e with v in [2^(e-1), 2^e), limited so that 2^(9 - e) and its inverse are normal.
__device__ __forceinline__ int scale_exponent(float v) {
  int e = 0;
  if (v > 0.0f && v < __builtin_inff()) (void)__builtin_frexpf(v, &e);
  return e < -100 ? -100 : (e > 100 ? 100 : e);
}

// Two fp32 values times sc as fp16 parts: x sc = hi + lo, 22 significant bits.
__device__ __forceinline__ void split2_f16(float x0, float x1, float sc, uint32_t& hi, uint32_t& lo) {
  const f32x2 x = f32x2{x0 * sc, x1 * sc};
  const f16x2 xh = __builtin_convertvector(x, f16x2);
  hi = __builtin_bit_cast(uint32_t, xh);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[0] - (float)xh[0], x[1] - (float)xh[1]}, f16x2));
}

}  // namespace spectra_dev
