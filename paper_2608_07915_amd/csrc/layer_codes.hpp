// Kept-group tables and code operands shared by the per-layer kernels.
#pragma once
#include "device_common.hpp"

namespace spectra_dev {

constexpr int LG = 64;  // latent group size of the per-layer geometry
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;

// Kept groups of a per-layer stream in slot order (slot k: group, width, first payload
// word), then the dropped groups; built by the first wavefront of a workgroup in LDS, one
// group per lane (one load latency instead of a serial walk over the width table).
struct LayerTable {
  int grp[16], b[16], pay[16];
  int n_kept;  // kept groups: grp[0 .. n_kept); dropped ones follow in grp
  int used;    // record words used
  int ok;      // every width in [0, 8]
};
__device__ __forceinline__ void layer_table(const uint8_t* __restrict__ bits_s, int ng, int lane, LayerTable& t) {
  const int b = lane < ng ? bits_s[lane] : 0;
  const uint32_t kept = (uint32_t)__ballot(b > 0), below = (1u << (lane & 31)) - 1u;
  const bool ok = __ballot(b > 8) == 0;
  const int n = __popc(kept);
  int words = 0, before = 0;  // payload words of all groups, of the groups before this lane's
#pragma unroll
  for (int g = 0; g < 16; ++g) {
    const int bg = __builtin_amdgcn_readlane(b, g);
    before += g < lane ? 2 * bg : 0;
    words += 2 * bg;
  }
  if (lane < ng) {
    const int rank = __popc(kept & below);
    const int k = b > 0 ? rank : n + lane - rank;
    t.grp[k] = lane;
    t.b[k] = b;
    t.pay[k] = n + before;
  }
  if (lane == 0) {
    t.n_kept = n;
    t.used = n + words;
    t.ok = ok ? 1 : 0;
  }
}

// ---------------------------------------------------------------------------
// Codes of one token as fp16 matrix operands. Half h of a 64-code group at width B is
// the B payload words w[0 .. B) holding codes 32h + j, j < 32. Codes j and j + 16 lie B
// 16-bit halves apart at the same bit offset, so joining half i with half i + B puts
// them at the same offset of the two halves of one register, and one shift and one mask
// serve both; OR-ing in the exponent of 1024 and subtracting 1024 + 2^(B-1) (both
// exact) gives the two as fp16 integers centered on 0. About 1.6 instructions per code
// against 2.5 for single extraction and conversion. Operand element 2i + e of K step k
// is code 4k + i + 16e: the other operand is laid out to match (code_position).
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
// Place of group coefficient c (< 64) in the K order of codes_f16: K step k, lane half h
// and element e read place 32h + 8k + e.
__host__ __device__ constexpr int code_position(int c) { return (c & 32) + 2 * (c & 15) + ((c >> 4) & 1); }

}  // namespace spectra_dev
