// Decode-step attention over per-layer latents (App. E, Mode B; the latent spans all
// KV heads of a layer, d = n_kv_heads x 128, groups of 64). For query head h on KV head
// kv, k_t[kv rows] = (c_t + m_K) V_K[kv rows]^T, so the score is c_t . q~_h plus a
// constant that cancels in the softmax, with q~_h = q_h V_K[kv rows] a d-dimensional
// latent query; the output is (sum_t p_t c^V_t / sum_t p_t + m_V) V_V[kv rows]^T.
// Every query head reads the same per-token record, so one tile of records serves all
// heads of a sequence. With the square-root split (Eq. gsvd) the cached coordinate is
// c'_j = c_j f_j: the keys' 1 / f_j folds into the latent query (q~'_j = q~_j / f_j) and
// the values' sums are divided by f_j before m_V is added.
//
//   layer_qprep_kernel    q~ (scale and log2 e folded in) and its per-group sums;
//   layer_scores_kernel   scores of all heads for a chunk of 64-token tiles: codes
//                         (exact in fp16) times q~ as two fp16 parts, one kept group at a
//                         time, the token's scale and zero point applied after; chunk max;
//   layer_values_kernel   p = exp2(s - max over its two chunks), then per kept value group
//                         sum_t p_t s_t q_t on v_mfma_f32_16x16x32_bf16 (weights as two
//                         bf16 parts, codes of eight consecutive tokens read from the
//                         word-major tile) and sum_t p_t z_t;
//   layer_combine_kernel  softmax max and sum over the chunks, the chunk partials' sum,
//                         divided by it, plus m_V;
//   layer_rotate_kernel   applies V_V[kv rows]^T.
#include "device_common.hpp"
#include "kernels.hpp"
#include "attn_common.hpp"
#include "layer.hpp"
#include "layer_codes.hpp"
#include "splits.hpp"

namespace spectra_dev {

constexpr int LA_H = 32;     // query heads per sequence (at most)
constexpr int LA_ROW = 68;   // words per staged record row (64 tokens + pad)
constexpr int LA_WMAX = 128;  // record words per tensor
// record words per tile staged through registers: the kernels are instantiated for
// records of at most 64 words and of at most LA_WMAX words
__host__ __device__ constexpr int la_prefetch_words(int W) { return W <= 64 ? 64 : LA_WMAX; }

__device__ __forceinline__ bool layer_bits_ok(const uint8_t* __restrict__ bits_s, int ng, int W) {
  int used = 0;
  for (int g = 0; g < ng; ++g) {
    const int b = bits_s[g];
    if (b > 8) return false;
    if (b > 0) used += 1 + 2 * b;
  }
  return used <= W;
}

// ---------------------------------------------------------------------------
// q~[b][h][j] = scale log2(e) sum_i q[b][h][i] V_K[b][kv 128 + i][j] on kept groups
// ---------------------------------------------------------------------------
// grid (heads, sequences, d / 256): thread (coefficient j, quarter of the 128 rows), all its
// 32 loads in flight at once; four groups per workgroup
__global__ __launch_bounds__(1024) void layer_qprep_kernel(LayerAttnArgs a) {
  __shared__ float qv[128];
  __shared__ float part[4][256];
  __shared__ int slot_of[16];  // kept rank of each group
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, jj = tid & 255, quarter = tid >> 8;
  const int d = a.d, ng = d / 64;
  const int j = 256 * blockIdx.z + jj;
  const int kv = h / (a.n_q_heads / a.n_kv_heads);
  const uint8_t* bits_s = a.bits_k + (int64_t)b * ng;
  const bool kept = j < d && bits_s[j >> 6] > 0;
  const float* V = a.basis_k + (int64_t)b * d * d + (int64_t)(kv * 128 + 32 * quarter) * d + (j < d ? j : 0);
  float v[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = V[(int64_t)i * d];
  if (tid < ng) {
    int n = 0;
    for (int g = 0; g < tid; ++g) n += bits_s[g] > 0 ? 1 : 0;
    slot_of[tid] = n;
  }
  if (tid < 128) {
    const int64_t qi = ((int64_t)b * a.n_q_heads + h) * 128 + tid;
    qv[tid] = (a.q_f32 ? reinterpret_cast<const float*>(a.q)[qi] : bf2f(reinterpret_cast<const uint16_t*>(a.q)[qi])) *
              a.scale_log2;
  }
  __syncthreads();
  float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 32; ++i) sum[i & 3] = __builtin_fmaf(qv[32 * quarter + i], v[i], sum[i & 3]);
  part[quarter][jj] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
  __syncthreads();
  if (tid >= 256) return;
  float acc = kept ? (part[0][jj] + part[1][jj]) + (part[2][jj] + part[3][jj]) : 0.0f;
  if (kept && a.lscale_k) acc /= a.lscale_k[(int64_t)b * d + j];
  if (kept) {
    const int g = j >> 6;
    // fp16 parts for the score pass, at the group's kept slot
    const _Float16 hi = (_Float16)acc;
    const _Float16 lo = (_Float16)(acc - (float)hi);
    uint16_t* qh = a.qh + (int64_t)b * 2 * LA_H * d;
    const int place = 64 * slot_of[g] + code_position(j & 63);
    qh[(int64_t)h * d + place] = __builtin_bit_cast(uint16_t, hi);
    qh[(int64_t)(LA_H + h) * d + place] = __builtin_bit_cast(uint16_t, lo);
  }
  // group sums: a wavefront's 64 coefficients are one group (the score pass reads kept groups only)
  const float s = wave_sum_lane63(acc);
  if ((tid & 63) == 63 && j < d) a.qsum[((int64_t)b * a.n_q_heads + h) * 16 + (j >> 6)] = s;
}

// ---------------------------------------------------------------------------
// Scores
// ---------------------------------------------------------------------------
// Sixteen wavefronts per workgroup, each walking its own 32-token blocks over all kept
// slots (v_mfma_f32_32x32x16_f16: rows = 32 heads, columns = tokens): the latent queries
// sit in LDS as two fp16 parts, a token's payload words go from memory to registers two
// slots ahead and become operands there, so nothing is exchanged between wavefronts and
// the loop has no barrier. Scores of a tile are written as [head][64 tokens].
// For a 131k-token 1024-wide layer at 8x: eight wavefronts with the codes extracted from
// staged record rows 61 us; each wavefront holding two slots' queries in registers and the
// slots' sums meeting in LDS per tile 42 us (two wavefronts per SIMD, half of the time
// waiting for records); this form 33 us.
constexpr int LA_SW = 16;      // wavefronts per score workgroup
constexpr int LA_QP = LG + 8;  // fp16 per staged query row

__global__ __launch_bounds__(64 * LA_SW, 4) void layer_scores_kernel(LayerAttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t qa[16][2][LA_H][LA_QP];  // [slot][part][head][place]
  __shared__ __attribute__((aligned(16))) float qs[16][LA_H];  // [slot][head]: sums of the latent query over the slot's group
  __shared__ float wmax[LA_SW][LA_H];
  __shared__ LayerTable tab;
  const int chunk = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int h = lane >> 5, col = lane & 31;
  const int d = a.d, ng = d / 64, Hq = a.n_q_heads, Wk = a.Wk;
  if (wave == 0) layer_table(a.bits_k + (int64_t)b * ng, ng, lane, tab);
  __syncthreads();
  const int nk = __builtin_amdgcn_readfirstlane(tab.ok && tab.used <= Wk ? tab.n_kept : 0);
  const int tl = lane & 15;
  const int slot_b = tl < nk ? tab.b[tl] : 0, slot_pay = tl < nk ? tab.pay[tl] : 0;
  auto of_slot = [](int table, int slot) { return __builtin_amdgcn_readlane(table, slot); };

  const int64_t n_tiles = (a.n_tokens + 63) >> 6, n_blocks = (a.n_tokens + 31) >> 5;
  const int64_t blk0 = (int64_t)chunk * a.tiles_per_chunk * 2 + wave;
  int64_t blk_end = ((int64_t)chunk + 1) * a.tiles_per_chunk * 2;
  if (blk_end > n_blocks) blk_end = n_blocks;
  const uint32_t* kp = a.packed_k + (int64_t)b * a.t_cap * Wk + col;
  uint32_t words[2][8], meta[2] = {0u, 0u};  // slots in flight
  int w_slot = 0;
  int64_t w_blk = blk0;
  auto next_words = [&](int par) {  // past the last block its words are read again
    const int64_t bl = w_blk < blk_end ? w_blk : blk_end - 1;
    const uint32_t* src = kp + (bl >> 1) * (64 * (int64_t)Wk) + 32 * (bl & 1);
    const int bw = of_slot(slot_b, w_slot), pay = of_slot(slot_pay, w_slot);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < bw) words[par][i] = src[(pay + h * bw + i) * 64];
    meta[par] = src[w_slot * 64];
    if (++w_slot == nk) {
      w_slot = 0;
      w_blk += LA_SW;
    }
  };
  if (nk > 0 && blk0 < blk_end) {
    next_words(0);
    next_words(1);
  }
  for (int e = tid; e < 16 * LA_H; e += 64 * LA_SW) {
    const int sl = e >> 5, hd = e & 31;
    qs[sl][hd] = (hd < Hq && sl < nk) ? a.qsum[((int64_t)b * Hq + hd) * 16 + tab.grp[sl]] : 0.0f;
  }
  // 16-byte pieces: piece pc of row (part, head); rows of heads past n_q_heads are zero
#pragma unroll 4
  for (int e = tid; e < 2 * LA_H * 16 * 8; e += 64 * LA_SW) {
    const int pc = e & 127, row = e >> 7, part = row >> 5, hd = row & 31;
    if (pc < 8 * nk) {
      u32x4 v = u32x4{0u, 0u, 0u, 0u};
      if (hd < Hq) v = *reinterpret_cast<const u32x4*>(a.qh + ((int64_t)(2 * b + part) * LA_H + hd) * d + 8 * pc);
      *reinterpret_cast<u32x4*>(&qa[pc >> 3][part][hd][8 * (pc & 7)]) = v;
    }
  }
  uint32_t magic = 0x64006400u;  // exponent of 1024 in both halves, in a VGPR
  asm volatile("" : "+v"(magic));
  float mloc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) mloc[i] = -__builtin_inff();
  f32x16 S = {};
  int64_t blk = blk0;
  int slot = 0;
  // scores of block blk: lane (h, col) holds heads 8q + 4h + r of token col
  auto finish_block = [&]() {
    const int64_t t = 32 * blk + col;
    const bool valid = t < a.n_tokens;
    float* dst = a.scores + ((int64_t)b * n_tiles + (blk >> 1)) * Hq * 64 + 32 * (blk & 1) + col;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int hd = 8 * (i >> 2) + 4 * h + (i & 3);
      if (hd < Hq && valid) {
        dst[64 * hd] = S[i];
        mloc[i] = __builtin_fmaxf(mloc[i], S[i]);
      }
    }
    S = f32x16{};
    blk += LA_SW;
    slot = 0;
  };
  auto step = [&](auto pc) {
    constexpr int par = decltype(pc)::value;
    const int bw = of_slot(slot_b, slot);
    f16x8 cod[4];
    with_bits(bw, [&](auto bc) {
      constexpr int B = decltype(bc)::value;
      uint32_t Z[8];
      join_halves<B>(words[par], Z);
#pragma unroll
      for (int k = 0; k < 4; ++k) cod[k] = codes_f16<B>(Z, k, magic);
    });
    const float st = h2f(meta[par]), zc = __builtin_fmaf(st, (float)(1 << (bw - 1)), h2f(meta[par] >> 16));  // codes are centered
    next_words(par);
    f32x16 g = {};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int p = 0; p < 2; ++p)
        g = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const f16x8*>(&qa[slot][p][col][32 * h + 8 * k]), cod[k], g, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 qv = *reinterpret_cast<const f32x4*>(&qs[slot][8 * q + 4 * h]);
#pragma unroll
      for (int r = 0; r < 4; ++r) S[4 * q + r] = __builtin_fmaf(st, g[4 * q + r], __builtin_fmaf(zc, qv[r], S[4 * q + r]));
    }
    asm volatile("" : "+v"(S));  // summed here, not with every product alive across the next branch
    if (++slot == nk) finish_block();
  };
  __syncthreads();  // queries and group sums
  if (nk == 0) {
    while (blk < blk_end) finish_block();
  } else if (blk < blk_end) {
    const int64_t steps = (blk_end - blk + LA_SW - 1) / LA_SW * nk;
    for (int64_t i = 0; i < steps; i += 2) {
      step(std::integral_constant<int, 0>{});
      if (i + 1 < steps) step(std::integral_constant<int, 1>{});
    }
  }
  // chunk maxima of every head
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    float m = mloc[i];
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) m = __builtin_fmaxf(m, __shfl_xor(m, o));
    if (col == 0) wmax[wave][8 * (i >> 2) + 4 * h + (i & 3)] = m;
  }
  __syncthreads();
  if (tid < Hq) {
    float m = -__builtin_inff();
    for (int w = 0; w < LA_SW; ++w) m = __builtin_fmaxf(m, wmax[w][tid]);
    a.cmax[((int64_t)b * a.n_chunks + chunk) * Hq + tid] = m;
  }
}

// ---------------------------------------------------------------------------
// Values: one workgroup per (two score chunks, block of 16 query heads, half of the kept
// slots, sequence); wavefront w takes kept value slot w or w + 8. The halves are workgroups
// of their own so that two fit a CU (four wavefronts per SIMD): with both slots in one
// wavefront 61 us for a 131072-token 1024-wide layer at 8x, now 58 us (codes taken one
// at a time from staged rows, both slots: 91 us). At 131104 tokens the chunks are 18 tiles
// instead of 16 on 456 workgroups instead of 512: 67 us. The form for more than 64 words
// spills 15 registers (60 bytes of scratch a lane).
// ---------------------------------------------------------------------------
// Lane (kg, c16) of a product over 32 tokens supplies coefficients 4 c16 .. 4 c16 + 3 of
// the group for tokens 8 kg .. 8 kg + 7: four codes are at most 32 adjacent bits, so one
// window per token (from two staged record words) holds the operands of four products.
// Widths below 8 enter as 1 + c 2^-b, the code in the top b bits of the 7-bit mantissa
// under the exponent of 1.0; a second product against -1.5 turns that into c 2^-b - 1/2
// tile by tile (the sums stay near 0; the zero points take the 2^(b-1) s_t back). CLS 0: b in {1, 2, 4} (the four codes never cross a word); 1: b = 3; 2: b in
// {5, 6, 7} (codes 2 and 3 from the window shifted by 2b); 3: b = 8 (exact integers).
template <int CLS>
__device__ __forceinline__ void value_codes4(const uint32_t* __restrict__ rec, int pay, int b, int c16, int tk0, uint32_t magic,
                                             u32x4 (&r)[4]) {
  const int bit = 4 * c16 * b, sh = bit & 31;
  const uint32_t* src = rec + (pay + (bit >> 5)) * LA_ROW + tk0;
  const u32x4 l0 = *reinterpret_cast<const u32x4*>(src), l1 = *reinterpret_cast<const u32x4*>(src + 4);
  if constexpr (CLS == 3) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t y0 = i < 2 ? l0[2 * i] : l1[2 * i - 4], y1 = i < 2 ? l0[2 * i + 1] : l1[2 * i - 3];
#pragma unroll
      for (int c = 0; c < 4; ++c) r[c][i] = int_to_bf16_pair((y0 >> (8 * c)) & 0xFFu, (y1 >> (8 * c)) & 0xFFu);
    }
  } else {
    // z: the 16 bits from the window's start, of two tokens; a code at bit o of both
    // halves is rotated to bits 7 - b .. 6 (bits of the other half and wrapped ones land
    // outside the mask)
    const uint32_t M = ((1u << b) - 1u) << (7 - b), MM = M | (M << 16);
    uint32_t z[4], z2[4];
    int o = 0;
    if constexpr (CLS == 0) {  // two bytes from byte sh / 8; what is left of the offset (b = 1) goes to the rotation
      const uint32_t k = (uint32_t)sh >> 3, sel = __builtin_amdgcn_perm(k, k, 0u) + 0x05040100u;
      o = sh & 7;
      z[0] = __builtin_amdgcn_perm(l0[1], l0[0], sel);
      z[1] = __builtin_amdgcn_perm(l0[3], l0[2], sel);
      z[2] = __builtin_amdgcn_perm(l1[1], l1[0], sel);
      z[3] = __builtin_amdgcn_perm(l1[3], l1[2], sel);
    } else {
      // the next word is only needed when the window crosses into it; it is another staged
      // row at most (the one past the last is padding)
      const u32x4 h0 = *reinterpret_cast<const u32x4*>(src + LA_ROW), h1 = *reinterpret_cast<const u32x4*>(src + LA_ROW + 4);
      uint32_t y[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = __builtin_amdgcn_alignbit(h0[e], l0[e], sh);
        y[4 + e] = __builtin_amdgcn_alignbit(h1[e], l1[e], sh);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[i] = __builtin_amdgcn_perm(y[2 * i + 1], y[2 * i], 0x05040100u);
        if constexpr (CLS == 2) z2[i] = __builtin_amdgcn_perm(y[2 * i + 1] >> (2 * b), y[2 * i] >> (2 * b), 0x05040100u);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t zz = CLS == 2 && c >= 2 ? z2[i] : z[i];
        const int oc = o + (CLS == 2 ? c & 1 : c) * b;
        r[c][i] = (rotr32(zz, (uint32_t)(32 + oc - (7 - b)) & 31u) & MM) | magic;
      }
  }
}

constexpr int LA_PX = 32;  // floats after a partial row's d value sums: zero-point sums of 16 groups, sum of the weights

template <int WP>
__global__ __launch_bounds__(512, 4) void layer_values_kernel(LayerAttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t rec[(WP + 1) * LA_ROW];  // + a row that windows may touch
  __shared__ __attribute__((aligned(16))) float pl[16 * LA_ROW];
  __shared__ float mh[LA_H];
  __shared__ LayerTable tab;
  const int chunk = blockIdx.x, hbk = blockIdx.y >> 1, half = blockIdx.y & 1, b = blockIdx.z;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, kg = lane >> 4, c16 = lane & 15;
  const int d = a.d, ng = d / 64, Wv = a.Wv, Hq = a.n_q_heads;
  const bool key_ok = layer_bits_ok(a.bits_k + (int64_t)b * ng, ng, a.Wk);
  if (wave == 0) layer_table(a.bits_v + (int64_t)b * ng, ng, lane, tab);
  if (tid < LA_H) {
    float m = -__builtin_inff();
    if (tid < Hq)
      for (int c = 2 * chunk; c < 2 * chunk + 2 && c < a.n_chunks; ++c)
        m = __builtin_fmaxf(m, a.cmax[((int64_t)b * a.n_chunks + c) * Hq + tid]);
    // where every score of the two chunks is -inf the weights are exp2(-inf - 0) = 0, not NaN
    mh[tid] = m == -__builtin_inff() ? 0.0f : m;
  }
  if (tid < LA_ROW) rec[WP * LA_ROW + tid] = 0u;
  __syncthreads();
  const bool ok = key_ok && tab.ok && tab.used <= Wv;
  const int nk = __builtin_amdgcn_readfirstlane(ok ? tab.n_kept : 0);
  if (half && nk <= 8) return;  // uniform over the workgroup
  f32x4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int sl = 8 * half + wave;
  const int sb = sl < nk ? __builtin_amdgcn_readfirstlane(tab.b[sl]) : 0;
  const int sp = sl < nk ? __builtin_amdgcn_readfirstlane(tab.pay[sl]) : 0;
  // sums over this wavefront's slot and the lane's tokens: weights, weights times zero point
  float wsum = 0.0f, zsum = 0.0f;

  const int64_t n_tiles = (a.n_tokens + 63) >> 6;
  const int64_t t_begin = (int64_t)chunk * a.v_tiles_per_chunk;
  const int64_t t_end = t_begin + a.v_tiles_per_chunk < n_tiles ? t_begin + a.v_tiles_per_chunk : n_tiles;
  const uint32_t* vp = a.packed_v + (int64_t)b * a.t_cap * Wv;
  constexpr int PF = 64 * WP / 512;            // record rows per wavefront and tile
  constexpr int PS = 16 * 64 / 512;            // scores per thread and tile
  uint32_t pre[PF];
  float spre[PS], lacc[PS], mref[PS];
#pragma unroll
  for (int i = 0; i < PS; ++i) {
    lacc[i] = 0.0f;
    mref[i] = mh[16 * hbk + wave + 8 * i];
  }
  // the rows of this workgroup's slots: metadata row per slot, payload rows [row_lo, row_hi)
  const int row_lo = half ? __builtin_amdgcn_readfirstlane(tab.pay[8]) : nk;
  const int row_hi = !half && nk > 8 ? __builtin_amdgcn_readfirstlane(tab.pay[8]) : Wv;
  // wavefront w stages rows w, w + 8, .. (lane = token). Slots past n_tokens in the last
  // tile get weight 0; their metadata words are staged as 0 so that whatever the cache
  // holds there (a NaN scale or zero-point) never enters the products (0 * NaN would reach
  // every head through the MFMA).
  auto load_tile = [&](int64_t tt) {
    const bool in = tt * 64 + lane < a.n_tokens;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int row = wave + 8 * i;
      if (row < nk ? (row >> 3) == half : (row >= row_lo && row < row_hi)) {
        pre[i] = vp[tt * 64 * Wv + 64 * row + lane];
        if (row < nk && !in) pre[i] = 0u;
      }
    }
#pragma unroll
    for (int i = 0; i < PS; ++i) {
      const int h = 16 * hbk + wave + 8 * i;
      spre[i] = h < Hq && in ? a.scores[(((int64_t)b * n_tiles + tt) * Hq + h) * 64 + lane] : -__builtin_inff();
    }
  };
  uint32_t magic = 0x3F803F80u;  // exponent of 1.0 in both halves, in a VGPR
  asm volatile("" : "+v"(magic));
  const bf16x8 mid = as_bf16x8(u32x4{0xBFC0BFC0u, 0xBFC0BFC0u, 0xBFC0BFC0u, 0xBFC0BFC0u});  // -1.5
  if (ok && t_begin < t_end) load_tile(t_begin);
  for (int64_t tt = (ok ? t_begin : t_end); tt < t_end; ++tt) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int row = wave + 8 * i;
      if (row < nk ? (row >> 3) == half : (row >= row_lo && row < row_hi)) rec[row * LA_ROW + lane] = pre[i];
    }
#pragma unroll
    for (int i = 0; i < PS; ++i) {
      const float pv = __builtin_amdgcn_exp2f(spre[i] - mref[i]);
      pl[(wave + 8 * i) * LA_ROW + lane] = pv;
      lacc[i] += pv;
    }
    __syncthreads();
    if (tt + 1 < t_end) load_tile(tt + 1);
    if (sb > 0) {
      auto body = [&](auto cls) {
        constexpr int CLS = decltype(cls)::value;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const int tk0 = 32 * ks + 8 * kg;
          // weights p_t s_t of head 16 hbk + c16 for tokens tk0 .. tk0 + 7 as two bf16 parts:
          // the fp32 exponent range (p_t s_t spans many decades below 1) and 16 significant
          // bits (relative error below 2^-17 per weight; a third part changed the output by
          // 1e-6 relative and cost 7% of the call)
          bf16x8 wp[2];
          {
            const float* pr = pl + c16 * LA_ROW + tk0;
            const f32x4 p0 = *reinterpret_cast<const f32x4*>(pr), p1 = *reinterpret_cast<const f32x4*>(pr + 4);
            const uint32_t* mr = rec + sl * LA_ROW + tk0;
            const u32x4 m0 = *reinterpret_cast<const u32x4*>(mr), m1 = *reinterpret_cast<const u32x4*>(mr + 4);
            u32x4 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float pa = e < 2 ? p0[2 * e] : p1[2 * e - 4], pc = e < 2 ? p0[2 * e + 1] : p1[2 * e - 3];
              const uint32_t ma = e < 2 ? m0[2 * e] : m1[2 * e - 4], mc = e < 2 ? m0[2 * e + 1] : m1[2 * e - 3];
              const f32x2 w = f32x2{pa * h2f(ma), pc * h2f(mc)};
              wsum += w[0];
              wsum += w[1];
              zsum = __builtin_fmaf(pa, h2f(ma >> 16), zsum);
              zsum = __builtin_fmaf(pc, h2f(mc >> 16), zsum);
              const uint32_t hb = __builtin_bit_cast(uint32_t, __builtin_convertvector(w, bf16x2));
              const f32x2 rest = f32x2{w[0] - __uint_as_float(hb << 16), w[1] - __uint_as_float(hb & 0xFFFF0000u)};
              hi[e] = hb;
              lo[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, bf16x2));
            }
            wp[0] = as_bf16x8(hi);
            wp[1] = as_bf16x8(lo);
          }
          u32x4 cv[4];
          value_codes4<CLS>(rec, sp, sb, c16, tk0, magic, cv);
#pragma unroll
          for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
              acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[q], as_bf16x8(cv[cb]), acc[cb], 0, 0, 0);
            if constexpr (CLS != 3)
#pragma unroll
              for (int cb = 0; cb < 4; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[q], mid, acc[cb], 0, 0, 0);
          }
        }
      };
      if (sb == 8)
        body(std::integral_constant<int, 3>{});
      else if (sb == 3)
        body(std::integral_constant<int, 1>{});
      else if (sb <= 4)
        body(std::integral_constant<int, 0>{});
      else
        body(std::integral_constant<int, 2>{});
    }
  }
  // partials: lane holds rows (heads 16 hbk + 4 kg + j) of coefficients 4 c16 .. 4 c16 + 3
  float* pb = a.part + ((int64_t)b * a.nv_chunks + chunk) * Hq * (d + LA_PX);
  if (sb > 0) {
    const float vs = sb < 8 ? (float)(1 << sb) : 1.0f;  // codes below 8 bits entered as c 2^-b - 1/2
    const int grp = __builtin_amdgcn_readfirstlane(tab.grp[sl]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int h = 16 * hbk + 4 * kg + j;
      if (h < Hq)
        *reinterpret_cast<f32x4*>(pb + (int64_t)h * (d + LA_PX) + 64 * grp + 4 * c16) =
            f32x4{acc[0][j] * vs, acc[1][j] * vs, acc[2][j] * vs, acc[3][j] * vs};
    }
  }
  // wavefront w: sums of the weights of heads 16 hbk + w + 8 i over its 64 token lanes
#pragma unroll
  for (int i = 0; i < PS; ++i) {
    const int h = 16 * hbk + wave + 8 * i;
    const float l = wave_sum_lane63(lacc[i]);
    if (half == 0 && lane == 63 && h < Hq) pb[(int64_t)h * (d + LA_PX) + d + 16] = l;
  }
  // lane (kg, c16) holds its tokens' share of head 16 hbk + c16
  float zt = __builtin_fmaf(wsum, sb > 0 && sb < 8 ? (float)(1 << (sb - 1)) : 0.0f, zsum);
  zt += __shfl_xor(zt, 16);
  zt += __shfl_xor(zt, 32);
  if (sb > 0 && kg == 0 && 16 * hbk + c16 < Hq) pb[(int64_t)(16 * hbk + c16) * (d + LA_PX) + d + tab.grp[sl]] = zt;
}

// ---------------------------------------------------------------------------
// Combine: c[j] = (sum over value chunks of exp2(their maximum - overall maximum) times
// (coefficient sums + zero-point sums)) / softmax sum + m_V[j], written over q~ (no longer
// needed); grid (heads, sequences, d / 64 groups). The softmax maximum over the
// score chunks and the weights' sum over the value chunks are taken by every workgroup itself (one maximum per chunk).
// ---------------------------------------------------------------------------
constexpr int LA_CHUNKS = spectra::N_CU;  // score chunks per sequence (at most)

__global__ __launch_bounds__(256) void layer_combine_kernel(LayerAttnArgs a) {
  // thread -> (coefficient 64 z + (tid & 63), every fourth chunk from tid >> 6): four short
  // chains of loads instead of one long one, summed in LDS in a fixed order
  __shared__ float ps[4][64], cm[LA_CHUNKS], cf[LA_CHUNKS / 2 + 64], red[3][4];
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int d = a.d, ng = d / 64, Hq = a.n_q_heads;
  const int j = 64 * blockIdx.z + (tid & 63), part = tid >> 6;
  const uint8_t* bv = a.bits_v + (int64_t)b * ng;
  const bool ok = layer_bits_ok(bv, ng, a.Wv) && layer_bits_ok(a.bits_k + (int64_t)b * ng, ng, a.Wk);
  const int g = j >> 6;  // one group per workgroup
  const bool kept = ok && bv[g] > 0;
  const int64_t cstride = (int64_t)Hq * (d + LA_PX);
  const float* pb = a.part + ((int64_t)b * a.nv_chunks * Hq + h) * (d + LA_PX);
  const float m = tid < a.n_chunks ? a.cmax[((int64_t)b * a.n_chunks + tid) * Hq + h] : -__builtin_inff();
  const float lv = ok && tid < a.nv_chunks ? pb[tid * cstride + d + 16] : 0.0f;
  const float zv = kept && tid < a.nv_chunks ? pb[tid * cstride + d + g] : 0.0f;
  cm[tid] = m;
  const float mw = wave_max_all(m);
  if ((tid & 63) == 0) red[0][part] = mw;
  __syncthreads();
  const float M = __builtin_fmaxf(__builtin_fmaxf(red[0][0], red[0][1]), __builtin_fmaxf(red[0][2], red[0][3]));
  float f = 0.0f;
  if (tid < LA_CHUNKS / 2) {
    const float mv = __builtin_fmaxf(cm[2 * tid], cm[2 * tid + 1]);
    f = mv != -__builtin_inff() ? __builtin_amdgcn_exp2f(mv - M) : 0.0f;
  }
  if (tid < LA_CHUNKS / 2 + 64) cf[tid] = f;  // 0 past the last chunk
  const float lw = wave_sum_lane63(f * lv), zw = wave_sum_lane63(f * zv);
  if ((tid & 63) == 63) {
    red[1][part] = lw;
    red[2][part] = zw;
  }
  __syncthreads();
  float s0 = 0.f, s1 = 0.f;
  if (kept) {
    // sixteen loads in flight; chunks past the last read it again with weight 0
    for (int c0 = __builtin_amdgcn_readfirstlane(part); c0 < a.nv_chunks; c0 += 64) {
      float x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int ch = c0 + 4 * i;
        x[i] = pb[(ch < a.nv_chunks ? ch : a.nv_chunks - 1) * cstride + j];
      }
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        s0 = __builtin_fmaf(cf[c0 + 4 * i], x[i], s0);
        s1 = __builtin_fmaf(cf[c0 + 4 * i + 4], x[i + 1], s1);
      }
    }
  }
  ps[part][tid & 63] = s0 + s1;
  __syncthreads();
  if (tid < 64) {
    const float L = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    const float inv_l = L > 0.0f ? 1.0f / L : 0.0f;
    float c = 0.0f;
    if (kept && M != -__builtin_inff())  // no score above -inf: no weight, the output is the mean's
      c = (((ps[0][tid] + ps[1][tid]) + (ps[2][tid] + ps[3][tid])) + ((red[2][0] + red[2][1]) + (red[2][2] + red[2][3]))) *
          inv_l;
    if (a.lscale_v) c /= a.lscale_v[(int64_t)b * d + j];
    a.qt[((int64_t)b * Hq + h) * d + j] = c + a.mean_v[(int64_t)b * d + j];
  }
}

// ---------------------------------------------------------------------------
// Inverse rotation: out[i] = sum_j c[j] V_V[kv 128 + i][j]; grid (heads, sequences, 16):
// workgroup z takes rows 8 z .. 8 z + 7, two per wavefront, each row read by the whole
// wavefront (d / 64 values per lane), then a wavefront sum
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void layer_rotate_kernel(LayerAttnArgs a) {
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, Hq = a.n_q_heads;
  const int kv = h / (Hq / a.n_kv_heads);
  const float* cfv = a.qt + ((int64_t)b * Hq + h) * d;
  // every load before the first use: columns past d read column `lane` again, times 0
  float cl[16], v[2][16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int j = 64 * k + lane < d ? 64 * k + lane : lane;
    cl[k] = 64 * k < d ? cfv[j] : 0.0f;
#pragma unroll
    for (int r = 0; r < 2; ++r)
      v[r][k] = a.basis_v[(int64_t)b * d * d + (int64_t)(kv * 128 + 8 * (int)blockIdx.z + 2 * wave + r) * d + j];
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (64 * k < d) acc = __builtin_fmaf(cl[k], v[r][k], acc);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) a.out[((int64_t)b * Hq + h) * 128 + 8 * blockIdx.z + 2 * wave + r] = acc;
  }
}

}  // namespace spectra_dev

namespace spectra {
using namespace spectra_dev;

// Value pass: two score chunks per workgroup and head block, so its softmax reference is
// the larger of their two maxima.
static int32_t layer_value_chunks(int32_t batch, int64_t n_tokens, int32_t* tiles_per_chunk) {
  const Split s = layer_score_split(batch, (n_tokens + 63) / 64);
  *tiles_per_chunk = 2 * s.tiles_per_chunk;
  return (s.n_chunks + 1) / 2;
}

// Sized for the most chunks that any token count up to n_tokens is split into, so a workspace
// taken for a longer cache serves every shorter one.
size_t layer_attention_ws_floats(int32_t batch, int32_t n_q_heads, int32_t d, int64_t n_tokens) {
  const int64_t n_tiles = (n_tokens + 63) / 64, nch = layer_score_chunks(batch, n_tiles), nv = (nch + 1) / 2;
  const int64_t B = batch, H = n_q_heads;
  auto r64 = [](int64_t n) { return (n + 63) / 64 * 64; };  // 256-byte aligned sections
  return (size_t)(r64(B * H * d) + r64(B * LA_H * d) + r64(B * H * 16) + r64(B * H * n_tiles * 64) + r64(B * nch * H) +
                  r64(B * nv * H * (d + LA_PX)));
}

void layer_attention_ws_layout(LayerAttnArgs& a, float* ws) {
  const Split s = layer_score_split(a.batch, (a.n_tokens + 63) / 64);
  a.n_chunks = s.n_chunks;
  a.tiles_per_chunk = s.tiles_per_chunk;
  a.nv_chunks = layer_value_chunks(a.batch, a.n_tokens, &a.v_tiles_per_chunk);
  const int64_t B = a.batch, H = a.n_q_heads;
  auto r64 = [](int64_t n) { return (n + 63) / 64 * 64; };
  a.qt = ws;
  a.qh = reinterpret_cast<uint16_t*>(a.qt + r64(B * H * a.d));  // 2 x 32 x d halves = 32 x d floats
  a.qsum = a.qt + r64(B * H * a.d) + r64(B * LA_H * a.d);
  a.scores = a.qsum + r64(B * H * 16);
  a.cmax = a.scores + r64(B * H * ((a.n_tokens + 63) / 64 * 64));
  a.part = a.cmax + r64(B * a.n_chunks * H);
}

hipError_t launch_layer_attention(const LayerAttnArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(layer_qprep_kernel, dim3(a.n_q_heads, a.batch, (a.d + 255) / 256), dim3(1024), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(layer_scores_kernel, dim3(a.n_chunks, a.batch), dim3(64 * LA_SW), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (la_prefetch_words(a.Wv) > 64)
    hipLaunchKernelGGL(layer_values_kernel<LA_WMAX>, dim3(a.nv_chunks, 4, a.batch), dim3(512), 0, st, a);
  else
    hipLaunchKernelGGL(layer_values_kernel<64>, dim3(a.nv_chunks, 4, a.batch), dim3(512), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(layer_combine_kernel, dim3(a.n_q_heads, a.batch, a.d / 64), dim3(256), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(layer_rotate_kernel, dim3(a.n_q_heads, a.batch, 16), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace spectra
