// How the kernels' grids split tokens over workgroups (plain C++17, shared by the launchers
// and host-side checks). A workgroup that starts when the others end costs a whole round, so
// no grid is rounded up past what the card's CUs hold at once.
#pragma once
#include <cstdint>

namespace spectra {

constexpr int64_t N_CU = 256;  // compute units of the card

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Chunk c of a token range: tiles [c tiles_per_chunk, (c + 1) tiles_per_chunk).
struct Split {
  int32_t tiles_per_chunk, n_chunks;
};
inline Split split_tiles(int64_t n_tiles, int64_t tiles_per_chunk) {
  return Split{(int32_t)tiles_per_chunk, (int32_t)ceil_div(n_tiles, tiles_per_chunk)};
}

// ---------------------------------------------------------------------------
// Reconstruction of per-head records
// ---------------------------------------------------------------------------
constexpr int DECODE_WAVES = 8;  // wavefronts of a workgroup, each rebuilding its own units
struct DecodeGrid {
  int32_t per_stream;  // workgroups per stream
  int32_t waves;       // of a workgroup
  bool half_tiles;     // units of 32 tokens instead of 64
};

// One round of workgroups, one per CU (LDS and registers), each of which splits its stream's
// basis once; rounded up instead (12 streams: 264 workgroups), 32000 tokens of 12 streams took
// 60 us, now 43, of 40 streams 184, now 162. Units of 64 tokens, but of 32 as long as no
// wavefront then has more than one: the chain through one unit sets the time of short windows
// (eight heads at 12x: 500 tokens 13.7 us by whole tiles in one workgroup per stream, now 10.6,
// and 12.3 with four wavefronts sharing a tile; 4000 tokens 15.0, now 12.5, and 14.3; 8192 at
// 8x 18.3 and 17.1, beyond which halves would be a second round). Up to two tiles: a workgroup of four
// wavefronts, of which a CU holds two (264 streams of 64 tokens: 24 us, now 16; eight streams
// 12.8, now 11.3).
inline DecodeGrid decode_grid(int64_t n_streams, int64_t n_tiles) {
  if (n_tiles <= 2) return DecodeGrid{1, 4, true};
  const int64_t n = N_CU > n_streams ? N_CU / n_streams : 1;
  const bool half = 2 * n_tiles <= n * DECODE_WAVES;
  const int64_t most = half ? 2 * n_tiles : ceil_div(n_tiles, DECODE_WAVES);
  return DecodeGrid{(int32_t)(n < most ? n : most), DECODE_WAVES, half};
}

// ---------------------------------------------------------------------------
// Workspace of the per-head attention calls, in chunks per (sequence, KV head)
// ---------------------------------------------------------------------------
// What one call has room for: the larger of chunks of at least 16 tiles for 768 workgroups
// over all tiles but the last, plus that tile's, and chunks of at least four tiles for 512. Not
// monotone in the tiles: a longer cache can have longer and fewer chunks.
inline int32_t attention_max_chunks(int64_t groups, int64_t n_tiles) {
  const int64_t body = n_tiles > 0 ? n_tiles - 1 : 0;
  int64_t tpc = ceil_div(body, ceil_div(768, groups)), rope_tpc = ceil_div(n_tiles, ceil_div(2 * N_CU, groups));
  if (tpc < 16) tpc = 16;
  if (rope_tpc < 4) rope_tpc = 4;
  const int64_t scan = ceil_div(body, tpc) + 1, rope = ceil_div(n_tiles, rope_tpc);
  return (int32_t)(scan > rope ? scan : rope);
}

// The most of those over all caches of up to n_tiles tiles, so that a workspace taken for the
// longest cache serves every shorter one: chunks of their smallest length, as long as there
// are no more of them than wanted.
inline int32_t attention_workspace_chunks(int64_t groups, int64_t n_tiles) {
  const int64_t want = ceil_div(768, groups), rope_want = ceil_div(2 * N_CU, groups);
  const int64_t body = ceil_div(n_tiles - 1, 16), rope = ceil_div(n_tiles, 4);
  int64_t n = (body < want ? body : want) + 1;
  if (n < rope && n < rope_want) n = rope < rope_want ? rope : rope_want;
  return (int32_t)n;
}

// ---------------------------------------------------------------------------
// Latent attention scan
// ---------------------------------------------------------------------------
// Split for a scan kernel of which a CU holds per_cu workgroups of four wavefronts, a tile per
// wavefront and step. The last tile is a chunk of its own (in a decode step its workgroup also
// appends the new token); the others come in chunks of at least 8 tiles. The cuts set the order
// of the sums, and a decode step returns what attention alone does over the same records, so
// they depend on nothing that differs between the two calls.
//
// In a decode step the append is the longest chain of a short cache, and more workgroups only
// take its CU's time: there the shortest chunks of 8, 12 or 16 tiles that leave every
// workgroup a CU of its own (eight heads at 12x, 20000 tokens: 23.3 us by 320 workgroups, 21.1
// by 216; at 8x 24.3 and 22.5). Attention alone would rather have more of them (eight heads at
// 8x, 28000 tokens: 21.0 us by 440 workgroups, 23.1 by 232, which take 25.3 and 23.5 for the
// step; 128 groups of 1000 tokens 25.8 and 30.1, the step 42.4 and 40.3). The heavier a tile,
// the less the append counts. `weight` is the head quads times the words of both records: above
// 24 (four heads at 4x, seven at 8x) chunks of 16 lose against more workgroups (two sequences of
// 12000 tokens at 4x 30.1 and 29.1 us), above 32 (seven heads at 4x) so do all (32768 tokens
// 36.8 and 35.6).
//
// Otherwise as many chunks as fill the slots: a few workgroups beyond the slots start when the
// others end and nearly double the scan's time (32k tokens at 4x, 512 slots: 520 workgroups
// 33.5 us, 352 workgroups 26.5), so the count is rounded down, over the fewest rounds of
// workgroups that come out 85% full. The last tiles' workgroups need slots too. Up to eight
// groups the other chunks make room. Above, they are the last of the grid, and queue when the
// slot that one takes would cost the other chunks a tile per wavefront (64 groups at 8x, 16000
// tokens: the step 54.6 us with a queue, 45.1 without; 30000: 66.8 and 65.0, attention alone
// 59.3 and 63.2).
// Calls against chunks of at least 16 tiles for 768 workgroups: 32k tokens at 4x 35.5 -> 31.0
// us, seven heads over 65k tokens 38.0 -> 34.2, 1000 tokens 21.9 -> 17.6; equal from 48k to
// 131k tokens at 8x.
constexpr int SCAN_WAVES = 4;
inline Split scan_split(int64_t groups, int64_t n_tiles, int per_cu, int weight) {
  const int64_t body = n_tiles - 1, slots = N_CU * per_cu;
  if (body < 1) return Split{1, 1};
  for (int64_t t = 8; t <= (weight <= 24 ? 16 : weight <= 32 ? 12 : 0); t += SCAN_WAVES)
    if (groups * (ceil_div(body, t) + 1) <= N_CU) return Split{(int32_t)t, (int32_t)ceil_div(body, t) + 1};
  int64_t n = 0;
  for (int64_t rounds = 1; rounds <= 4; ++rounds) {
    n = rounds * slots / groups;
    if (n * groups * 100 >= 85 * rounds * slots) break;
  }
  if (n > 1 && (groups <= 8 || body < SCAN_WAVES * n * n)) --n;
  const int64_t cap = attention_max_chunks(groups, n_tiles) - 1, most = ceil_div(body, 8);
  if (n > cap) n = cap;
  if (n > most) n = most;
  if (n < 1) n = 1;
  int64_t tpc = ceil_div(body, n);
  if (tpc < 16) tpc = ceil_div(tpc, SCAN_WAVES) * SCAN_WAVES;  // whole steps
  return Split{(int32_t)tpc, (int32_t)ceil_div(body, tpc) + 1};
}

// ---------------------------------------------------------------------------
// Reconstruction of per-layer records
// ---------------------------------------------------------------------------
// Workgroups per channel block and stream (`blocks` of these in all), walking the token ranges
// in turn: at most one workgroup per CU (LDS) over all blocks, and no more than the longest
// walk needs. Rounded up instead, three 1024-wide streams made 264 workgroups and 65k tokens
// took 1114 us, now 760; one 768-wide stream 224 and 149.
inline int64_t layer_decode_split(int64_t ranges, int64_t blocks) {
  const int64_t n = blocks < N_CU ? N_CU / blocks : 1, each = ceil_div(ranges, n);
  return ceil_div(ranges, each);
}

// ---------------------------------------------------------------------------
// Per-layer attention
// ---------------------------------------------------------------------------
// Chunks of the score pass per sequence (the value pass takes two of them at a time): at most
// one workgroup per CU (LDS) over all sequences, at least two tiles each. Rounded up instead,
// three sequences made 258 workgroups and 65k tokens took 215 us, now 165; 24 sequences of 4000
// tokens 325 and 291.
constexpr int LAYER_MIN_TILES = 2;
inline int64_t layer_chunks_wanted(int64_t batch) { return batch < N_CU ? N_CU / batch : 1; }
inline Split layer_score_split(int64_t batch, int64_t n_tiles) {
  const int64_t tpc = ceil_div(n_tiles, layer_chunks_wanted(batch));
  return split_tiles(n_tiles, tpc < LAYER_MIN_TILES ? LAYER_MIN_TILES : tpc);
}
// The most that any cache of up to n_tiles tiles is split into.
inline int64_t layer_score_chunks(int64_t batch, int64_t n_tiles) {
  const int64_t most = ceil_div(n_tiles, LAYER_MIN_TILES), want = layer_chunks_wanted(batch);
  return most < want ? most : want;
}

// ---------------------------------------------------------------------------
// Rotary attention
// ---------------------------------------------------------------------------
enum class RopeKernel { WAVE, FOUR, EIGHT };  // a tile per wavefront, per four, per eight wavefronts
struct RopeSplit {
  RopeKernel kernel;
  Split split;
};
constexpr int ROPE_WAVE_TILES = 8;  // tiles that a workgroup of the wavefront kernel takes at a time

// Split for a kernel of which a CU holds per_cu workgroups, each taking `at_once` tiles of its
// chunk at a time: as many chunks of at least four tiles as one round of workgroups holds, or
// two rounds of one workgroup per CU, whichever has fewer steps (the preparation counts as one
// and a third). With the count rounded up, 12 groups (28 query heads on 4 KV heads, batch 3)
// made 264 workgroups for 256 CUs: 32k tokens 155 us, now 90; eight KV heads at batch 5 220 us,
// now 150 (four wavefronts per tile, before: 105 and 338).
inline Split rope_chunks(int64_t groups, int64_t n_tiles, int per_cu, int at_once) {
  Split best{};
  int64_t best_cost = 0;
  for (int rounds = 1; rounds * per_cu <= 2; ++rounds) {
    int64_t n = N_CU * per_cu * rounds / groups;
    if (n < 1) n = 1;
    int64_t tpc = ceil_div(n_tiles, n);
    if (tpc < 4) tpc = 4;
    const Split s = split_tiles(n_tiles, tpc);
    const int64_t cost = ceil_div(s.n_chunks * groups, N_CU * per_cu) * (4 + 3 * ceil_div(tpc, at_once));
    if (rounds == 1 || cost < best_cost) {
      best_cost = cost;
      best = s;
    }
  }
  return best;
}

// Up to four query heads per KV head with records of at most 16 words and up to eight with at
// most 8 words fit the wavefront kernel's LDS, and it is the faster one (131k tokens, four
// heads: 119 us against 183; 65k, seven heads: 65 against 76; 1000 tokens: 29 against 37), but
// for seven heads where its chunks have nine or ten tiles: the second step of eight wavefronts
// then has one or two at work (57.5 us against 56.5 at 9 tiles and one sequence, 63 against 58
// at 10 and four). The other shapes of up to 16 words take the four-wavefront kernel (two
// workgroups per CU), wider records the eight-wavefront kernel.
inline RopeSplit rope_split(int64_t groups, int n_qh, int words, int64_t n_tiles) {
  const bool few = n_qh <= 4;
  if (words <= (few ? 16 : 8)) {
    const Split s = rope_chunks(groups, n_tiles, 1, ROPE_WAVE_TILES);
    const int t = s.tiles_per_chunk;
    if (few || t <= ROPE_WAVE_TILES || t > ROPE_WAVE_TILES + 2) return RopeSplit{RopeKernel::WAVE, s};
  }
  if (!few && words <= 16) return RopeSplit{RopeKernel::FOUR, rope_chunks(groups, n_tiles, 2, 1)};
  return RopeSplit{RopeKernel::EIGHT, rope_chunks(groups, n_tiles, 1, 1)};
}

}  // namespace spectra
