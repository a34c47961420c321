// Kept-group tables of the per-layer kernels and the K order of their code operands.
#pragma once
#include "code_operands.hpp"

namespace spectra_dev {

constexpr int LG = 64;  // latent group size of the per-layer geometry

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

// Place of group coefficient c (< 64) in the K order of codes_f16, lane half h holding codes
// 32h .. 32h + 31: K step k, half h and element e read place 32h + 8k + e.
__host__ __device__ constexpr int code_position(int c) { return (c & 32) + 2 * (c & 15) + ((c >> 4) & 1); }

}  // namespace spectra_dev
