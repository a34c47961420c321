// Per-layer cross-head latent (Sec. 3.1 applied to a layer's whole KV vector, the
// geometry of Sec. 4.1 and App. F: d = d_kv = n_kv_heads x 128, latent groups of
// g = 64 coefficients). A stream is one (sequence, layer, tensor) T x d matrix; the
// record format is the per-head one with 64-coefficient groups (one metadata word
// per kept group, then 2b payload words per kept group at b bits).
//
// Kernels:
//   layer_gram_kernel     fp64 second moment x^T x of every stream, split over
//                         token ranges (deterministic partial sums), 64 x 64 tiles;
//   layer_moments_kernel  sums the partials in a fixed order and adds the column sums;
//   layer_encode_kernel   c = x V - m on v_mfma_f32_32x32x16_bf16 (bf16 tokens exact,
//                         the fp32 basis as three bf16 parts staged through LDS), then
//                         per token and kept group fp16 zero-point and scale, codes,
//                         packing; one workgroup per (256 tokens, kept group, stream);
//   layer_decode_kernel   x_hat = sum_G (s_tG q_tG + z_tG 1) V_G^T + m V^T: codes
//                         unpacked in registers, the basis columns of a group as two
//                         fp16 parts in LDS, the group's per-token scale applied after
//                         its product; persistent workgroups of 128 channels.
#include "attn_common.hpp"
#include "device_common.hpp"
#include "kernels.hpp"
#include "layer.hpp"
#include "layer_codes.hpp"
#include "splits.hpp"

namespace spectra_dev {

// Kept group `slot` of a per-layer stream (widths bits_s[0..ng)): group index, width
// and first payload word; also the number of kept groups and the record words used.
struct LayerSlot {
  int grp, b, pay, n_kept, used;
  bool ok;  // every width in [0, 8]
};
__device__ __forceinline__ LayerSlot layer_slot(const uint8_t* __restrict__ bits_s, int ng, int slot) {
  LayerSlot r{-1, 0, 0, 0, 0, true};
  int n = 0, payw = 0;
  for (int g = 0; g < ng; ++g) {
    const int b = bits_s[g];
    if (b > 8) r.ok = false;
    if (b > 0) {
      if (n == slot) {
        r.grp = g;
        r.b = b;
        r.pay = payw;  // relative to the end of the metadata words
      }
      ++n;
      payw += 2 * b;
    }
  }
  r.n_kept = n;
  r.pay += n;
  r.used = n + payw;
  return r;
}

// ---------------------------------------------------------------------------
// Moments
// ---------------------------------------------------------------------------
template <bool F32IN>
__device__ __forceinline__ double load_x(const void* x, int64_t i) {
  if constexpr (F32IN)
    return (double)reinterpret_cast<const float*>(x)[i];
  else
    return (double)bf2f(reinterpret_cast<const uint16_t*>(x)[i]);
}

// partial[s][kc] = [sum over tokens [kc * ck, min(n, (kc + 1) ck)) of x_t^T x_t (d x d),
// then the column sums over the same tokens (d)], 64 x 64 output tile per workgroup,
// 16-token steps staged in LDS, 4 x 4 outputs per thread. The workgroups of the first
// tile column also sum their 64 channels: each thread over the tokens it stages (every
// 16th), then the 16 shares of a channel in order.
template <bool F32IN>
__global__ __launch_bounds__(256) void layer_gram_kernel(LayerGramArgs g) {
  __shared__ double As[16][65];
  __shared__ double Bs[16][65];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int i0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
  const int s = blockIdx.z / g.k_split, kc = blockIdx.z % g.k_split;
  const int64_t t_begin = (int64_t)kc * g.chunk_tokens;
  const int64_t t_end = t_begin + g.chunk_tokens < g.n ? t_begin + g.chunk_tokens : g.n;
  const int64_t xb = (int64_t)s * g.stream_stride;
  const bool col_sums = blockIdx.y == 0;  // uniform over the workgroup
  double csum[4] = {0.0, 0.0, 0.0, 0.0};
  double acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = 0.0;
  for (int64_t t0 = t_begin; t0 < t_end; t0 += 16) {
    // 16 tokens x 64 channels of each operand: thread -> (token tid >> 4, channels 4 (tid & 15) ..)
    {
      const int tk = tid >> 4, c4 = 4 * (tid & 15);
      const int64_t t = t0 + tk;
      const bool in = t < t_end;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double xa = in ? load_x<F32IN>(g.x, xb + t * g.token_stride + i0 + c4 + e) : 0.0;
        As[tk][c4 + e] = xa;
        Bs[tk][c4 + e] = in ? load_x<F32IN>(g.x, xb + t * g.token_stride + j0 + c4 + e) : 0.0;
        if (col_sums) csum[e] += xa;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      double a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = As[k][ty + 16 * q];
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = Bs[k][tx + 16 * q];
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[p][q] = __builtin_fma(a[p], b[q], acc[p][q]);
    }
    __syncthreads();
  }
  const int64_t dd = (int64_t)g.d * g.d;
  double* out = g.partial + ((int64_t)s * g.k_split + kc) * (dd + g.d);
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) out[(int64_t)(i0 + ty + 16 * p) * g.d + j0 + tx + 16 * q] = acc[p][q];
  if (col_sums) {
    const int tk = tid >> 4, c4 = 4 * (tid & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) As[tk][c4 + e] = csum[e];  // the loop ended with a barrier
    __syncthreads();
    if (tid < 64) {
      double cs = 0.0;
      for (int k = 0; k < 16; ++k) cs += As[k][tid];
      out[dd + i0 + tid] = cs;
    }
  }
}

// moments[s] = sum_kc partial[s][kc] ([d x d Gram, d column sums]), partials added in
// ascending kc.
template <bool F32IN>
__global__ __launch_bounds__(256) void layer_moments_kernel(LayerGramArgs g) {
  const int s = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t dd = (int64_t)g.d * g.d;
  double* mom = g.moments + (int64_t)s * (dd + g.d);
  if (e < dd + g.d) {
    const double* p = g.partial + (int64_t)s * g.k_split * (dd + g.d) + e;
    double acc = 0.0;
    for (int kc = 0; kc < g.k_split; ++kc) acc += p[kc * (dd + g.d)];
    mom[e] = acc;
  }
}

// ---------------------------------------------------------------------------
// Encode
// ---------------------------------------------------------------------------
// Workgroups of a one-dimensional grid over (token range, block) are dispatched to the
// eight XCDs in turn (workgroup i to XCD i mod 8). Numbering them i = 8 (nb r + blk) + x
// with token range 8 r + x puts every block of a range on the same XCD, close together
// in time, so that XCD's L2 serves the range's rows to all of them instead of every XCD
// fetching them from HBM. Ranges past the last one (the grid is rounded up to whole
// groups of eight) get range = -1.
__host__ __device__ constexpr unsigned xcd_major_grid(int n_ranges, int nb) { return 8u * (unsigned)nb * (unsigned)((n_ranges + 7) / 8); }
__device__ __forceinline__ void xcd_major_block(int n_ranges, int nb, int& range, int& blk) {
  const int i = (int)blockIdx.x, x = i & 7, j = i >> 3;
  blk = j % nb;
  range = 8 * (j / nb) + x;
  if (range >= n_ranges) range = -1;
}

constexpr int LE_TOK = 256;       // tokens per workgroup (eight wavefronts of 32)
constexpr int LE_KC = 64;         // basis rows per staged chunk
constexpr int LE_KP = LE_KC + 8;  // bf16 per staged row (144-byte rows, 16-byte aligned)

// Row of the staged 64-row operand that holds group coefficient c: within each
// 32-row block, row r feeds coefficient 16 ((r >> 2) & 1) + (r & 3) + 4 (r >> 3), so
// that after the 32x32 product lane half h holds coefficients 16h .. 16h + 15.
__device__ __forceinline__ int le_row(int c) {
  const int cc = c & 31;
  return 32 * (c >> 5) + (cc & 3) + 4 * (cc >> 4) + 8 * ((cc >> 2) & 3);
}

__global__ __launch_bounds__(512, 4) void layer_encode_kernel(LayerEncodeArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t vs[3][64][LE_KP];
  const int s = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: the staging rows are scalar
  const int d = a.d, ng = d / LG;
  int range, slot;
  xcd_major_block((int)((a.n + LE_TOK - 1) / LE_TOK), ng, range, slot);
  if (range < 0) return;
  const LayerSlot ks = layer_slot(a.bits + (int64_t)s * ng, ng, slot);
  const int64_t sbase = (int64_t)s * a.t_cap * a.W;
  const int64_t wg_tok = (int64_t)range * LE_TOK;
  if (!ks.ok || ks.used > a.W) return;  // width table inconsistent with the record: write nothing

  // words past the used ones are zero: written by the slot-0 workgroup
  if (slot == 0 && ks.used < a.W) {
    const int nw = a.W - ks.used;
    for (int e = tid; e < LE_TOK * nw; e += 512) {
      const int64_t i = wg_tok + (e % LE_TOK);
      if (i < a.n) a.packed[rec_word(sbase, a.t0 + i, a.W, ks.used + e / LE_TOK)] = 0u;
    }
  }
  if (slot >= ks.n_kept) return;  // uniform over the workgroup

  const int64_t i_tok = wg_tok + 32 * wave + col;
  const bool valid = i_tok < a.n;
  const int64_t i_ld = valid ? i_tok : a.n - 1;
  const uint16_t* xr = reinterpret_cast<const uint16_t*>(a.x) + (int64_t)s * a.stream_stride + i_ld * a.token_stride;
  const float* V = a.basis + (int64_t)s * d * d + LG * ks.grp;

  // staging map: thread -> (group coefficient sc, basis rows sk .. sk + 7 of the chunk)
  const int sc = tid & 63, sk = 8 * wave, srow = le_row(sc);
  float pre[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) pre[i] = V[(int64_t)(sk + i) * d + sc];
  u32x4 xb[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) xb[k] = *reinterpret_cast<const u32x4*>(xr + 16 * k + 8 * h);

  // Accumulation order, for fp32 accuracy over d up to 1024 terms: the products with
  // the basis' high bf16 part are summed per 64-row chunk and the chunk sums added
  // into the running totals; the two low parts (2^-8 and 2^-16 of the value) go to a
  // separate accumulator whose rounding is correspondingly small.
  f32x16 acc0 = {}, acc1 = {}, sm0 = {}, sm1 = {};
  const int nk = d / LE_KC;
  for (int kc = 0; kc < nk; ++kc) {
    {
      uint32_t p0[8], p1[8], p2[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) split3(pre[i], p0[i], p1[i], p2[i]);
      *reinterpret_cast<u32x4*>(&vs[0][srow][sk]) = u32x4{pack2(p0[0], p0[1]), pack2(p0[2], p0[3]), pack2(p0[4], p0[5]), pack2(p0[6], p0[7])};
      *reinterpret_cast<u32x4*>(&vs[1][srow][sk]) = u32x4{pack2(p1[0], p1[1]), pack2(p1[2], p1[3]), pack2(p1[4], p1[5]), pack2(p1[6], p1[7])};
      *reinterpret_cast<u32x4*>(&vs[2][srow][sk]) = u32x4{pack2(p2[0], p2[1]), pack2(p2[2], p2[3]), pack2(p2[4], p2[5]), pack2(p2[6], p2[7])};
    }
    __syncthreads();
    if (kc + 1 < nk) {
#pragma unroll
      for (int i = 0; i < 8; ++i) pre[i] = V[(int64_t)((kc + 1) * LE_KC + sk + i) * d + sc];
    }
    f32x16 ch0 = {}, ch1 = {};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bf16x8 xk = as_bf16x8(xb[k]);
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const bf16x8 a0 = as_bf16x8(*reinterpret_cast<const u32x4*>(&vs[p][col][16 * k + 8 * h]));
        const bf16x8 a1 = as_bf16x8(*reinterpret_cast<const u32x4*>(&vs[p][32 + col][16 * k + 8 * h]));
        if (p == 0) {
          ch0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, xk, ch0, 0, 0, 0);
          ch1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, xk, ch1, 0, 0, 0);
        } else {
          sm0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, xk, sm0, 0, 0, 0);
          sm1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, xk, sm1, 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      acc0[i] += ch0[i];
      acc1[i] += ch1[i];
    }
    if (kc + 1 < nk) {
#pragma unroll
      for (int k = 0; k < 4; ++k) xb[k] = *reinterpret_cast<const u32x4*>(xr + (kc + 1) * LE_KC + 16 * k + 8 * h);
    }
    __syncthreads();
  }

  // lane (h, col): coefficients 16h + i (acc0) and 32 + 16h + i (acc1) of token col. The
  // lane's token and half are recomputed here rather than held in registers across the loop.
  int tid_e = tid;
  asm volatile("" : "+v"(tid_e));
  const int he = (tid_e & 63) >> 5;
  const int64_t i_tok_e = wg_tok + 32 * wave + (tid_e & 31);
  const bool valid_e = i_tok_e < a.n;
  const int64_t i_ld_e = valid_e ? i_tok_e : a.n - 1;
  const float* mg = a.mean + (int64_t)s * d + LG * ks.grp;
  float c[32];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    c[i] = (acc0[i] + sm0[i]) - mg[16 * he + i];
    c[16 + i] = (acc1[i] + sm1[i]) - mg[32 + 16 * he + i];
  }
  if (a.lscale) {  // square-root split: the cached coordinate is (x V - m)_j f_j
    const float* fg = a.lscale + (int64_t)s * d + LG * ks.grp;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      c[i] *= fg[16 * he + i];
      c[16 + i] *= fg[32 + 16 * he + i];
    }
  }
  float lo = c[0], hi = c[0];
#pragma unroll
  for (int i = 1; i < 32; ++i) {
    lo = __builtin_fminf(lo, c[i]);
    hi = __builtin_fmaxf(hi, c[i]);
  }
  lo = __builtin_fminf(lo, __shfl_xor(lo, 32));
  hi = __builtin_fmaxf(hi, __shfl_xor(hi, 32));
  const int64_t base = rec_word(sbase, a.t0 + i_ld_e, a.W, 0);
  with_bits(ks.b, [&](auto bc) {
    constexpr int B = decltype(bc)::value;
    constexpr float LEV = (float)((1 << B) - 1);
    const uint32_t z16 = f2h_sat(lo);
    const float z = h2f(z16);
    const uint32_t s16 = f2h_sat(__builtin_fmaxf(hi - z, 0.0f) / LEV);
    const float sf = h2f(s16);
    const float rinv = sf > 0.0f ? 1.0f / sf : 0.0f;
    uint32_t q0[16], q1[16], P0[4], P1[4];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      q0[i] = (uint32_t)__builtin_fminf(__builtin_fmaxf(__builtin_rintf((c[i] - z) * rinv), 0.0f), LEV);
      q1[i] = (uint32_t)__builtin_fminf(__builtin_fmaxf(__builtin_rintf((c[16 + i] - z) * rinv), 0.0f), LEV);
    }
    pack16<B>(q0, P0);
    pack16<B>(q1, P1);
    if (he == 0 && valid_e) a.packed[base + (int64_t)slot * TILE] = s16 | (z16 << 16);
    store_payload<B>(a.packed, base, ks.pay, P0, he, valid_e);
    store_payload<B>(a.packed, base, ks.pay + B, P1, he, valid_e);
  });
}

// ---------------------------------------------------------------------------
// Decode (Mode A)
// ---------------------------------------------------------------------------
// One workgroup: 128 output channels, walking ranges of 256 tokens (wavefront w: 32 tokens x
// all 128 channels). What depends on the channels alone is computed once per workgroup:
// m V^T, the sums of the basis entries of each kept group, a power of two per channel that
// brings its largest entry near 1 and then one per group that brings its largest into [2^8, 2^9)
// (channels far weaker than a group's strongest keep their 22 bits). Then, per kept group of a range, the 128 x 64
// basis block goes to LDS as two fp16 parts (two buffers: the next block is split while
// this one is multiplied) and each lane turns its token's payload words into operands in
// registers:
//   out[ch][t] += s_t (sum_j V[ch][j] q'_tj), q' the codes centered on 0.
// Two fp16 parts of the scaled entries keep 22 bits and take two products where three bf16
// parts took three; centering the codes halves the magnitude of the fp32 sums, so the error
// against 64 bits went down (2.9e-7 -> 2.3e-7). The zero-point terms (z_t + 2^(b-1) s_t)
// sum_j V[ch][j] of all groups are one product over the slots per range (three bf16 parts
// each side), and m V^T is added last.
// The codes are the row operand and column c of channel block b is channel 4c + b, so every
// store of a wavefront is two whole 512-byte row pieces.
// A 131k-token 1024-wide layer at 8x: 1860 -> 481 us. The counters have the matrix cores busy
// 43% of the time and the vector ALU 42%; the wavefronts wait 29% of their cycles (the store
// bursts at a range's end, LDS inside a step) and 33% for their turn to issue. What was tried
// and is slower: a workgroup per range (720 us: its prologue and epilogue overlap nothing), 64
// tokens x 64 channels per wavefront (560 us, every code unpacked twice), 64 x 128 (490 to 520
// us, spills), four wavefronts with four times the registers (770 us).
constexpr int LD_CH = 128;     // channels per workgroup
constexpr int LD_NW = 8;       // wavefronts per workgroup
constexpr int LD_TOK = 32 * LD_NW;  // tokens per range
constexpr int LD_P = LG + 8;   // fp16 per LDS row (144 bytes: 16 rows on distinct banks)
constexpr int LD_RB = 33;      // rows from one 32-channel block to the next (the four blocks' rows of a write on distinct banks)
constexpr int LD_YP = 24;      // bf16 per row of the group sums (16 slots + pad)
constexpr int LD_ZP = 20;      // floats per row of the zero points (16 slots + pad)

__device__ __forceinline__ void split_row3(const float (&x)[8], bf16x8 (&p)[3]) {
  uint32_t p0[8], p1[8], p2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) split3(x[i], p0[i], p1[i], p2[i]);
  p[0] = as_bf16x8(u32x4{pack2(p0[0], p0[1]), pack2(p0[2], p0[3]), pack2(p0[4], p0[5]), pack2(p0[6], p0[7])});
  p[1] = as_bf16x8(u32x4{pack2(p1[0], p1[1]), pack2(p1[2], p1[3]), pack2(p1[4], p1[5]), pack2(p1[6], p1[7])});
  p[2] = as_bf16x8(u32x4{pack2(p2[0], p2[1]), pack2(p2[2], p2[3]), pack2(p2[4], p2[5]), pack2(p2[6], p2[7])});
}

template <bool SCALED>
__global__ __launch_bounds__(64 * LD_NW, 2) void layer_decode_kernel(LayerDecodeArgs a) {
  constexpr int NT = 64 * LD_NW;
  static_assert(NT == 4 * LD_CH, "a thread stages a quarter of a channel's 64 coefficients");
  __shared__ __attribute__((aligned(16))) uint16_t vl[2][2][4 * LD_RB][LD_P];  // [buffer][part][row][place]
  __shared__ __attribute__((aligned(16))) uint16_t yl[3][4 * LD_RB][LD_YP];    // [part][row][slot]: group sums
  __shared__ __attribute__((aligned(16))) float zl[LD_TOK][LD_ZP];         // [token][slot]: centered zero points
  __shared__ __attribute__((aligned(16))) float scl[LD_TOK];               // scales of the slot at hand
  __shared__ __attribute__((aligned(16))) float bias[LD_CH];
  __shared__ __attribute__((aligned(16))) float mean[1024];
  __shared__ __attribute__((aligned(16))) float rscale[LD_CH];  // of each channel: the inverse of its row's scale
  __shared__ int vexp[16];
  __shared__ LayerTable tab;
  // largest entry of each channel in a kept group; the basis blocks take its place afterwards
  float(*vmax)[LD_CH] = reinterpret_cast<float(*)[LD_CH]>(vl);
  static_assert(16 * LD_CH * sizeof(float) <= sizeof(vl), "maxima fit the basis blocks");
  const int s = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, ng = d / LG, nb = d / LD_CH;
  // channel block fastest: with eight blocks each XCD keeps one 128-row basis slice in its
  // L2 and streams the records, which are several times smaller than the rows they rebuild
  const int ch0 = (int)(blockIdx.x % (unsigned)nb) * LD_CH;
  const int64_t n_ranges = (a.n + LD_TOK - 1) / LD_TOK;
  const int64_t r_step = gridDim.x / (unsigned)nb;
  const int64_t sbase = (int64_t)s * a.t_cap * a.W;
  const float* Vs = a.basis + (int64_t)s * d * d;
  if (wave == 0) layer_table(a.bits + (int64_t)s * ng, ng, lane, tab);
  for (int i = tid; i < d; i += NT) mean[i] = a.mean[(int64_t)s * d + i];
  for (int i = tid; i < 3 * 4 * LD_RB * LD_YP / 2; i += NT) reinterpret_cast<uint32_t*>(yl)[i] = 0u;  // slots past the kept ones
  for (int i = tid; i < LD_TOK * LD_ZP; i += NT) reinterpret_cast<float*>(zl)[i] = 0.0f;
  __syncthreads();
  if (!tab.ok || tab.used > a.W) return;  // width table inconsistent with the record: write nothing
  const int n_kept = __builtin_amdgcn_readfirstlane(tab.n_kept);

  // staging share: channel row tid >> 2, group coefficients c0 .. c0 + 7 and c0 + 16 ..
  // c0 + 23, which are 16 consecutive places of the operand row
  const int ch = tid >> 2, sub = tid & 3, c0 = 32 * (sub >> 1) + 8 * (sub & 1);
  const int row = LD_RB * (ch & 3) + (ch >> 2);  // column c of 32-channel block b is channel 4c + b
  float v[16];
  auto load_v = [&](int g, float (&x)[16]) {
    const float* src = Vs + (int64_t)(ch0 + ch) * d + LG * g + c0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<f32x4*>(&x[4 * q]) = *reinterpret_cast<const f32x4*>(src + 16 * (q >> 1) + 4 * (q & 1));
  };
  // square-root split: c_hat_j / f_j folded into the basis columns
  auto scale_v = [&](int g, float (&x)[16]) {
    if constexpr (SCALED) {
      const float* f = a.lscale + (int64_t)s * d + LG * g + c0;
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] *= 1.0f / f[16 * (i >> 3) + (i & 7)];
    }
  };
  float rsc;  // this row's scale
  {
    float bsum = 0.0f, rmax = 0.0f, x[2][16];
    load_v(__builtin_amdgcn_readfirstlane(tab.grp[0]), x[0]);
    for (int k0 = 0; k0 < ng; k0 += 2) {  // d is a multiple of 128: an even number of groups
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = k0 + u, g = __builtin_amdgcn_readfirstlane(tab.grp[k]);
        load_v(__builtin_amdgcn_readfirstlane(tab.grp[k + 1 < ng ? k + 1 : k]), x[u ^ 1]);
        float(&xc)[16] = x[u];
#pragma unroll
        for (int i = 0; i < 16; ++i) bsum = __builtin_fmaf(mean[LG * g + c0 + 16 * (i >> 3) + (i & 7)], xc[i], bsum);
        if (k < n_kept) {
          scale_v(g, xc);
          float m = 0.0f, sum = 0.0f;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            sum += xc[i];
            m = __builtin_fmaxf(m, __builtin_fabsf(xc[i]));
          }
          sum += __shfl_xor(sum, 1);
          sum += __shfl_xor(sum, 2);
          uint32_t p0, p1, p2;
          split3(sum, p0, p1, p2);
          if (sub < 3) yl[sub][row][k] = (uint16_t)(sub == 0 ? p0 : sub == 1 ? p1 : p2);
          m = __builtin_fmaxf(m, __shfl_xor(m, 1));
          m = __builtin_fmaxf(m, __shfl_xor(m, 2));
          if (sub == 0) vmax[k][ch] = m;
          rmax = __builtin_fmaxf(rmax, m);
        }
      }
    }
    bsum += __shfl_xor(bsum, 1);
    bsum += __shfl_xor(bsum, 2);
    rsc = __builtin_ldexpf(1.0f, -row_exponent(rmax));
    if (sub == 0) {
      bias[ch] = bsum;
      rscale[ch] = 1.0f / rsc;
    }
  }
  __syncthreads();
  // every row is scaled to a largest entry near 1 and then every group to one in [2^8, 2^9)
#pragma unroll
  for (int u = 0; u < 16 / LD_NW; ++u) {
    const int k = wave + LD_NW * u;
    const float m = wave_max_all(__builtin_fmaxf(vmax[k][lane] / rscale[lane], vmax[k][64 + lane] / rscale[64 + lane]));
    if (lane == 0) vexp[k] = 9 - scale_exponent(m);  // read for kept slots only
  }
  __syncthreads();

  // slot tables, one slot per lane: read by v_readlane with a scalar slot, no memory access
  const int tl = lane & 15;
  const int slot_grp = tab.grp[tl < ng ? tl : 0], slot_b = tl < n_kept ? tab.b[tl] : 0, slot_pay = tl < n_kept ? tab.pay[tl] : 0;
  const int slot_exp = tl < n_kept ? vexp[tl] : 0;
  auto of_slot = [](int table, int slot) { return __builtin_amdgcn_readlane(table, slot); };

  // the group in v to buffer buf as two fp16 parts
  auto split_v = [&](int slot, int buf) {
    const float sc = __builtin_ldexpf(rsc, of_slot(slot_exp, slot));
    uint32_t hi[8], lo[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // coefficients c0 + i and c0 + 16 + i are neighbours in K
      split2_f16(v[i], v[8 + i], sc, hi[i], lo[i]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      *reinterpret_cast<u32x4*>(&vl[buf][0][row][16 * sub + 8 * q]) = u32x4{hi[4 * q], hi[4 * q + 1], hi[4 * q + 2], hi[4 * q + 3]};
      *reinterpret_cast<u32x4*>(&vl[buf][1][row][16 * sub + 8 * q]) = u32x4{lo[4 * q], lo[4 * q + 1], lo[4 * q + 2], lo[4 * q + 3]};
    }
  };

  // this lane's token of a range is row tw + col
  const int tw = 32 * wave;
  const uint32_t* rec = nullptr;
  uint32_t words[8], meta = 0u;
  int64_t range = blockIdx.x / (unsigned)nb;
  // record words of the next slot to come (all slots of a range, then the next range;
  // tokens past the last one read the last one)
  int w_slot = 0;
  int64_t w_range = range;
  auto next_words = [&]() {
    if (w_slot == 0) {
      const int64_t i = w_range * LD_TOK + tw + col;
      rec = a.packed + rec_word(sbase, a.t0 + (i < a.n ? i : a.n - 1), a.W, 0);
      w_range += r_step;
    }
    const int b = of_slot(slot_b, w_slot), pay = of_slot(slot_pay, w_slot);
    const uint32_t* src = rec + (pay + h * b) * TILE;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < b) words[i] = src[i * TILE];
    meta = rec[w_slot * TILE];
    w_slot = w_slot + 1 < n_kept ? w_slot + 1 : 0;
  };
  uint32_t magic = 0x64006400u;  // exponent of 1024 in both halves, in a VGPR
  asm volatile("" : "+v"(magic));
  // operands and centered zero point of the slot whose words are held (its scale is in LDS)
  f16x8 cod[4];
  float zc = 0.0f;
  int u_slot = 0;
  auto unpack = [&]() {
    const int bw = of_slot(slot_b, u_slot);
    with_bits(bw, [&](auto bc) {
      constexpr int B = decltype(bc)::value;
      uint32_t Z[8];
      join_halves<B>(words, Z);
#pragma unroll
      for (int k = 0; k < 4; ++k) cod[k] = codes_f16<B>(Z, k, magic);
    });
    const float sv = h2f(meta);
    scl[tw + col] = sv * __builtin_ldexpf(1.0f, -of_slot(slot_exp, u_slot));
    zc = __builtin_fmaf(sv, (float)(1 << (bw - 1)), h2f(meta >> 16));
    u_slot = u_slot + 1 < n_kept ? u_slot + 1 : 0;
  };
  f32x16 out[4];  // 32-channel blocks
  auto multiply = [&](int slot, int buf) {
    zl[tw + col][slot] = zc;
    f32x4 sr[4];  // scales of the rows of this lane's sums
#pragma unroll
    for (int q = 0; q < 4; ++q) sr[q] = *reinterpret_cast<const f32x4*>(&scl[tw + 8 * q + 4 * h]);
    // operands are read two K steps ahead and a channel block's sums are added while the
    // next block's products run
    constexpr int AHEAD = 2;
    f16x8 ah[AHEAD + 1], al[AHEAD + 1];
    f32x16 g[2];
    auto read_op = [&](int t) {
      const uint16_t* src = &vl[buf][0][LD_RB * (t >> 2) + col][32 * h + 8 * (t & 3)];
      ah[t % (AHEAD + 1)] = *reinterpret_cast<const f16x8*>(src);
      al[t % (AHEAD + 1)] = *reinterpret_cast<const f16x8*>(src + 4 * LD_RB * LD_P);
    };
    auto add_block = [&](int cb) {
#pragma unroll
      for (int i = 0; i < 16; ++i) out[cb][i] = __builtin_fmaf(sr[i >> 2][i & 3], g[cb & 1][i], out[cb][i]);
    };
#pragma unroll
    for (int t = 0; t < AHEAD; ++t) read_op(t);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int cb = t >> 2, k = t & 3;
      if (t + AHEAD < 16) read_op(t + AHEAD);
      if (k == 0) g[cb & 1] = f32x16{};
      g[cb & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cod[k], ah[t % (AHEAD + 1)], g[cb & 1], 0, 0, 0);
      g[cb & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cod[k], al[t % (AHEAD + 1)], g[cb & 1], 0, 0, 0);
      if (k == 3 && cb > 0) add_block(cb - 1);
    }
    add_block(3);
    __builtin_amdgcn_sched_group_barrier(0x100, 4 + 2 * AHEAD, 0);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      if (t + AHEAD < 16) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      if (t >= 5) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    }
    // the sums stay here (not sunk past the next blocks with all products alive)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) asm volatile("" : "+v"(out[cb]));
  };

  // Half of the wavefronts run the halves of a step in the opposite order (and unpack a
  // slot ahead), so that some split and unpack while others multiply.
  const bool ahead = wave >= LD_NW / 2;
  int buf = 0;
  if (n_kept > 0 && range < n_ranges) {
    next_words();
    const int g0 = of_slot(slot_grp, 0);
    load_v(g0, v);
    scale_v(g0, v);
    split_v(0, 0);
    const int g1 = of_slot(slot_grp, n_kept > 1 ? 1 : 0);
    load_v(g1, v);
    scale_v(g1, v);
    if (ahead) {
      unpack();
      next_words();
    }
    __syncthreads();
  }
  for (; range < n_ranges; range += r_step) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) out[cb] = f32x16{};
    // slot k of a range is multiplied from buffer buf while slot k + 1 is split into the
    // other and the basis block of slot k + 2 is loaded (modulo the kept slots: the next
    // range uses the same blocks); past the last range the prefetches repeat its words
    for (int slot = 0; slot < n_kept; ++slot) {
      const int s1 = slot + 1 < n_kept ? slot + 1 : 0, s2 = s1 + 1 < n_kept ? s1 + 1 : 0;
      if (ahead) multiply(slot, buf);
      split_v(s1, buf ^ 1);
      const int g2 = of_slot(slot_grp, s2);
      load_v(g2, v);
      unpack();
      next_words();
      if (!ahead) multiply(slot, buf);
      scale_v(g2, v);
      __syncthreads();
      buf ^= 1;
    }

    // zero-point terms over the slots: K element 8h + i is slot 8h + i
    float z[8];
    *reinterpret_cast<f32x4*>(&z[0]) = *reinterpret_cast<const f32x4*>(&zl[tw + col][8 * h]);
    *reinterpret_cast<f32x4*>(&z[4]) = *reinterpret_cast<const f32x4*>(&zl[tw + col][8 * h + 4]);
    bf16x8 zp[3];
    split_row3(z, zp);
    f32x16 y[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      bf16x8 yp[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) yp[p] = as_bf16x8(*reinterpret_cast<const u32x4*>(&yl[p][LD_RB * cb + col][8 * h]));
      y[cb] = f32x16{};
      y[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zp[2], yp[0], y[cb], 0, 0, 0);
      y[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zp[0], yp[2], y[cb], 0, 0, 0);
      y[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zp[1], yp[1], y[cb], 0, 0, 0);
      y[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zp[1], yp[0], y[cb], 0, 0, 0);
      y[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zp[0], yp[1], y[cb], 0, 0, 0);
      y[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zp[0], yp[0], y[cb], 0, 0, 0);
    }
    // lane (h, col): channels 4 col .. 4 col + 3 of tokens 8q + 4h + r: a store of the
    // wavefront is two whole 512-byte row pieces
    const f32x4 b4 = *reinterpret_cast<const f32x4*>(&bias[4 * col]), rs = *reinterpret_cast<const f32x4*>(&rscale[4 * col]);
    const int64_t i0 = range * LD_TOK + tw + 4 * h;
    float* o = a.out + ((int64_t)s * a.n + i0) * d + ch0 + 4 * col;
    const bool whole = range * LD_TOK + tw + 32 <= a.n;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = 8 * (i >> 2) + (i & 3);
      if (whole || i0 + r < a.n)
        *reinterpret_cast<f32x4*>(o + (int64_t)r * d) =
            f32x4{__builtin_fmaf(out[0][i], rs[0], y[0][i]) + b4[0], __builtin_fmaf(out[1][i], rs[1], y[1][i]) + b4[1],
                  __builtin_fmaf(out[2][i], rs[2], y[2][i]) + b4[2], __builtin_fmaf(out[3][i], rs[3], y[3][i]) + b4[3]};
    }
  }
}

}  // namespace spectra_dev

namespace spectra {
using namespace spectra_dev;

// Token split of the second moment: enough workgroups to fill the chip, chunks of
// at least 256 tokens.
void layer_gram_layout(int32_t d, int64_t n_streams, int64_t n_tokens, int32_t* k_split, int64_t* chunk_tokens) {
  const int64_t tiles = (int64_t)(d / 64) * (d / 64) * n_streams;
  int64_t ks = (2048 + tiles - 1) / tiles;
  const int64_t max_ks = (n_tokens + 255) / 256;
  ks = ks < 1 ? 1 : (ks > max_ks ? max_ks : ks);
  int64_t ct = (n_tokens + ks - 1) / ks;
  ct = (ct + 15) / 16 * 16;
  *chunk_tokens = ct;
  *k_split = (int32_t)((n_tokens + ct - 1) / ct);
}

hipError_t launch_layer_moments(const LayerGramArgs& g, bool f32_in, hipStream_t st) {
  const dim3 grid(g.d / 64, g.d / 64, g.n_streams * g.k_split);
  if (f32_in)
    hipLaunchKernelGGL(layer_gram_kernel<true>, grid, dim3(256), 0, st, g);
  else
    hipLaunchKernelGGL(layer_gram_kernel<false>, grid, dim3(256), 0, st, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t per = (int64_t)g.d * g.d + g.d;
  const dim3 grid2((unsigned)((per + 255) / 256), g.n_streams);
  if (f32_in)
    hipLaunchKernelGGL(layer_moments_kernel<true>, grid2, dim3(256), 0, st, g);
  else
    hipLaunchKernelGGL(layer_moments_kernel<false>, grid2, dim3(256), 0, st, g);
  return hipGetLastError();
}

hipError_t launch_layer_encode(const LayerEncodeArgs& a, hipStream_t st) {
  const dim3 grid(xcd_major_grid((int)((a.n + LE_TOK - 1) / LE_TOK), a.d / LG), 1, a.n_streams);
  hipLaunchKernelGGL(layer_encode_kernel, grid, dim3(512), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_layer_decode(const LayerDecodeArgs& a, hipStream_t st) {
  const int64_t nb = a.d / LD_CH;
  const dim3 grid((unsigned)(layer_decode_split((a.n + LD_TOK - 1) / LD_TOK, nb * a.n_streams) * nb), 1, a.n_streams);
  if (a.lscale)
    hipLaunchKernelGGL(layer_decode_kernel<true>, grid, dim3(64 * LD_NW), 0, st, a);
  else
    hipLaunchKernelGGL(layer_decode_kernel<false>, grid, dim3(64 * LD_NW), 0, st, a);
  return hipGetLastError();
}

}  // namespace spectra
