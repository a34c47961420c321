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

// Of a row whose largest entry is v: the exponent that it is scaled by, within 24 of 0 (so that
// sums and means in its scale stay finite).
__device__ __forceinline__ int row_exponent(float v) {
  const int e = v > 0.0f ? scale_exponent(v) : 0;
  return e < -24 ? -24 : (e > 24 ? 24 : e);
}

// Two fp32 values times sc as fp16 parts: x sc = hi + lo, 22 significant bits.
__device__ __forceinline__ void split2_f16(float x0, float x1, float sc, uint32_t& hi, uint32_t& lo) {
  const f32x2 x = f32x2{x0 * sc, x1 * sc};
  const f16x2 xh = __builtin_convertvector(x, f16x2);
  hi = __builtin_bit_cast(uint32_t, xh);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[0] - (float)xh[0], x[1] - (float)xh[1]}, f16x2));
}

// ---------------------------------------------------------------------------
// Basis of one KV head in LDS for a workgroup of NW (eight or four) wavefronts: row row_of(ch) of vl
// holds channel ch's entries of the kept groups as two fp16 parts, group slot sl scaled by
// the power of two that brings its largest entry into [2^8, 2^9) (exps[sl] is the inverse).
// With rscale, the row's entries, group sums and m V^T are first scaled by a power of two that
// brings its own largest entry near 1, and rscale[row] is the inverse: channels much weaker
// than a group's strongest keep their 22 bits (the second part ends 2^-34 below the group's
// largest entry; channels 10^5 times weaker came out with 5e-6 of error instead of 2e-7).
// coefficient c of a group at place 2 (c & 15) + (c >> 4). The same row of yl is the other
// operand of one product (K = 32, bf16) that gives a token's zero-point and mean terms,
// sum_sl zc_sl sum_j V[ch][j] + (m V^T)[ch]: slot sl has elements 8 sl .. 8 sl + 5 = parts 0 0 1
// 0 1 2 of the group's sum, against parts 0 1 0 2 1 0 of zc (zero_elements); elements 6,
// 7 and 14 hold the parts of m V^T, against ones. The caller synchronises afterwards.
// ---------------------------------------------------------------------------
constexpr int HB_NW = 8;         // wavefronts with a thread per (channel, group)
constexpr int HB_VP = D + 8;     // fp16 per basis row (272 bytes: 16 rows on distinct banks)
constexpr int HB_YP = 32 + 8;    // bf16 per row of group sums and m V^T
__host__ __device__ constexpr int hb_lds_bytes() { return (2 * D * HB_VP + D * HB_YP) * 2; }

template <int NW = HB_NW, typename RowFn>
__device__ __forceinline__ void stage_head_basis(const float* __restrict__ basis, const float* __restrict__ mean, const Kept& K,
                                                 int tid, uint16_t (*vl)[D][HB_VP], uint16_t (*yl)[HB_YP],
                                                 float (*vmax)[NG], float (&exps)[NG], float* rscale, RowFn&& row_of) {
  constexpr int IT = HB_NW / NW;  // channels per thread
  const int wave = tid >> 6, lane = tid & 63;
  const int g = tid & 3;
  float v[IT][32], sum[IT], bias[IT], rsc[IT], big = 0.0f;
  int slot = -1;  // kept slot of group g
#pragma unroll
  for (int sl = 0; sl < NG; ++sl) slot = (sl < K.n && K.grp[sl] == g) ? sl : slot;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const float* vr = basis + (int64_t)((tid >> 2) + 16 * NW * it) * D + G * g;
    const float* mr = mean + G * g;
    float m[32];
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<f32x4*>(&v[it][4 * i]) = *reinterpret_cast<const f32x4*>(vr + 4 * i);
#pragma unroll
    for (int i = 0; i < 32; ++i) m[i] = mr[i];
    sum[it] = bias[it] = 0.0f;
    float most = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      sum[it] += v[it][i];
      bias[it] = __builtin_fmaf(m[i], v[it][i], bias[it]);
      most = __builtin_fmaxf(most, __builtin_fabsf(v[it][i]));
    }
    bias[it] += __shfl_xor(bias[it], 1);
    bias[it] += __shfl_xor(bias[it], 2);
    rsc[it] = 1.0f;
    if (rscale != nullptr) {
      float rmax = slot >= 0 ? most : 0.0f;
      rmax = __builtin_fmaxf(rmax, __shfl_xor(rmax, 1));
      rmax = __builtin_fmaxf(rmax, __shfl_xor(rmax, 2));
      rsc[it] = __builtin_ldexpf(1.0f, -row_exponent(rmax));
      if (g == 0) rscale[row_of((tid >> 2) + 16 * NW * it)] = 1.0f / rsc[it];
    }
    big = __builtin_fmaxf(big, most * rsc[it]);
  }
#pragma unroll
  for (int o = 4; o < 64; o <<= 1) big = __builtin_fmaxf(big, __shfl_xor(big, o));
  if (lane < NG) vmax[wave][lane] = big;
  __syncthreads();
  int myexp = 0;
#pragma unroll
  for (int sl = 0; sl < NG; ++sl) {
    float mx = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) mx = __builtin_fmaxf(mx, vmax[w][K.grp[sl]]);
    const int e = __builtin_amdgcn_readfirstlane(9 - scale_exponent(mx));
    exps[sl] = __builtin_ldexpf(1.0f, -e);
    myexp = sl == slot ? e : myexp;
  }
  const float sc = __builtin_ldexpf(1.0f, myexp);
  int rank = 0;  // dropped group: its place among the slots past the kept ones
#pragma unroll
  for (int gg = 0; gg < NG; ++gg) {
    bool kept = false;
#pragma unroll
    for (int sl = 0; sl < NG; ++sl) kept = kept || (sl < K.n && K.grp[sl] == gg);
    rank += (!kept && gg < g) ? 1 : 0;
  }
  const int ys = slot >= 0 ? slot : K.n + rank;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int row = row_of((tid >> 2) + 16 * NW * it);
    if (slot >= 0) {
      // coefficients c and c + 16 are neighbours in K: place 2 (c & 15) + (c >> 4)
      uint32_t hi[16], lo[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) split2_f16(v[it][i], v[it][16 + i], sc * rsc[it], hi[i], lo[i]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<u32x4*>(&vl[0][row][G * slot + 8 * q]) = u32x4{hi[4 * q], hi[4 * q + 1], hi[4 * q + 2], hi[4 * q + 3]};
        *reinterpret_cast<u32x4*>(&vl[1][row][G * slot + 8 * q]) = u32x4{lo[4 * q], lo[4 * q + 1], lo[4 * q + 2], lo[4 * q + 3]};
      }
    }
    // row of the zero-point product: slot k has elements 8k .. 8k + 5 = group-sum parts
    // 0 0 1 0 1 2 (against z parts 0 1 0 2 1 0); elements 6, 7, 14 hold the parts of m V^T
    // (against ones); threads of dropped groups fill the slots past the kept ones with zeros
    uint32_t p0, p1, p2, b0, b1, b2;
    split3(slot >= 0 ? sum[it] * rsc[it] : 0.0f, p0, p1, p2);
    const float mv = bias[it] * rsc[it];
    split3(mv, b0, b1, b2);
    if (!(__builtin_fabsf(mv) < __builtin_inff())) {  // not finite: the first part alone (inf - inf is NaN)
      b0 = __float_as_uint(mv) >> 16;
      b1 = b2 = 0u;
    }
    const uint32_t tail = ys == 0 ? pack2(b0, b1) : ys == 1 ? pack2(b2, 0u) : 0u;
    *reinterpret_cast<u32x4*>(&yl[row][8 * ys]) = u32x4{pack2(p0, p0), pack2(p1, p0), pack2(p1, p2), tail};
  }
}

// The z side of that product for slot sl (< NG) of a token with metadata word m and width b
// (0: no such slot): the centered zero point zc = z + 2^(b-1) s in three bf16 parts.
__device__ __forceinline__ u32x4 zero_elements(uint32_t m, int b, uint32_t tail) {
  uint32_t z0 = 0u, z1 = 0u, z2 = 0u;
  if (b > 0) split3(__builtin_fmaf(h2f(m), __builtin_ldexpf(0.5f, b), h2f(m >> 16)), z0, z1, z2);
  return u32x4{pack2(z0, z1), pack2(z0, z2), pack2(z1, z0), tail};
}
// The ones against m V^T: slot 0 has two of its parts, slot 1 the third.
__device__ __forceinline__ uint32_t zero_tail(int sl) { return sl == 0 ? 0x3F803F80u : sl == 1 ? 0x00003F80u : 0u; }

}  // namespace spectra_dev
