// Host check of the grid splits (splits.hpp) over token counts and (sequence, KV head) groups:
// every tile in exactly one chunk and no chunk empty, no more chunks than a call's workspace
// holds, and no workgroups left over for a round of their own.
#include <cstdio>
#include <initializer_list>

#include "splits.hpp"

using namespace spectra;

static int bad = 0;
#define CHECK(cond, ...)                \
  do {                                  \
    if (!(cond)) {                      \
      if (++bad < 20) {                 \
        std::printf("%s: ", #cond);     \
        std::printf(__VA_ARGS__);       \
        std::printf("\n");              \
      }                                 \
    }                                   \
  } while (0)

static const int64_t GROUPS[] = {1, 2, 3, 4, 5, 8, 12, 16, 20, 24, 32, 40, 48, 64, 96, 100, 128, 160, 200, 256, 257, 300, 500, 512, 600, 900, 2000};

static void covers(const char* what, int64_t g, int64_t tiles, Split s) {
  CHECK(s.tiles_per_chunk > 0 && s.n_chunks > 0 && (int64_t)s.n_chunks * s.tiles_per_chunk >= tiles &&
            (int64_t)(s.n_chunks - 1) * s.tiles_per_chunk < tiles,
        "%s: %lld groups, %lld tiles: %d chunks of %d", what, (long long)g, (long long)tiles, s.n_chunks, s.tiles_per_chunk);
}

int main() {
  for (int64_t g : GROUPS)
    for (int64_t tiles = 1; tiles < 5000; tiles += tiles < 300 ? 1 : 7) {
      // one round of workgroups, none without a unit, halves only where no wavefront has two
      const DecodeGrid d = decode_grid(g, tiles);
      const int64_t units = d.half_tiles ? 2 * tiles : tiles, slots = d.waves == 4 ? 512 : 256;
      CHECK(d.per_stream >= 1 && d.per_stream <= (d.half_tiles ? units : ceil_div(units, d.waves)) && (d.per_stream * g <= slots || d.per_stream == 1), "decode: %lld streams, %lld tiles: %d",
            (long long)g, (long long)tiles, d.per_stream);
      CHECK(!d.half_tiles || units <= (int64_t)d.per_stream * d.waves, "decode: %lld streams, %lld tiles: a second half tile", (long long)g,
            (long long)tiles);
      CHECK(d.waves == 8 || (d.waves == 4 && d.half_tiles), "decode: %d wavefronts", d.waves);
    }
  for (int64_t g : GROUPS)
    for (int64_t ranges = 1; ranges < 3000; ++ranges) {
      const int64_t n = layer_decode_split(ranges, g);
      CHECK(n >= 1 && n <= ranges && (n * g <= 256 || n == 1) && (n == 1 || ceil_div(ranges, n - 1) > ceil_div(ranges, n)),
            "per-layer rows: %lld blocks, %lld ranges: %lld", (long long)g, (long long)ranges, (long long)n);
    }
  for (int64_t g : GROUPS) {
    int64_t layer_most = 0;
    for (int64_t tiles = 1; tiles < 9000; tiles += tiles < 800 ? 1 : 7) {
      const Split l = layer_score_split(g, tiles);
      const int64_t room = layer_score_chunks(g, tiles);
      covers("per layer", g, tiles, l);
      CHECK(l.n_chunks <= room && room >= layer_most && room <= 256 && (g > 256 || l.n_chunks * g <= 256),
            "per layer: %lld sequences, %lld tiles: %d chunks, room for %lld", (long long)g, (long long)tiles, l.n_chunks, (long long)room);
      layer_most = room;
    }
    int32_t most = 0;
    for (int64_t tiles = 1; tiles < 9000; tiles += tiles < 800 ? 1 : 7) {
      const int32_t cap = attention_max_chunks(g, tiles), ws = attention_workspace_chunks(g, tiles);
      CHECK(cap <= ws && ws >= most, "%lld groups, %lld tiles: %d, %d, %d", (long long)g, (long long)tiles, cap, ws, most);
      most = ws;
      for (int per_cu : {1, 2, 3})
        for (int weight : {10, 24, 25, 32, 33, 64}) {
          // the last tile is a chunk of its own
          const Split c = scan_split(g, tiles, per_cu, weight);
          if (tiles > 1)
            covers("scan", g, tiles - 1, Split{c.tiles_per_chunk, c.n_chunks - 1});
          else
            CHECK(c.n_chunks == 1, "scan: %d chunks of one tile", c.n_chunks);
          CHECK(c.n_chunks <= cap, "scan: %lld groups, %lld tiles: %d chunks, room for %d", (long long)g, (long long)tiles, c.n_chunks, cap);
          // a light shape's workgroups have a CU each where chunks of 16 tiles can do that
          CHECK(weight > 24 || g * (ceil_div(tiles - 1, 16) + 1) > 256 || g * c.n_chunks <= 256,
                "scan: %lld groups, %lld tiles: %d chunks", (long long)g, (long long)tiles, c.n_chunks);
          // up to eight groups: the last tiles' workgroups are held with the others
          CHECK(g > 8 || g * c.n_chunks <= 256 * per_cu, "scan: %lld groups, %lld tiles: %d chunks of %d", (long long)g, (long long)tiles,
                c.n_chunks, c.tiles_per_chunk);
        }
      for (int n_qh = 1; n_qh <= 8; n_qh += 3)
        for (int words : {4, 8, 9, 16, 17, 32}) {
          const RopeSplit r = rope_split(g, n_qh, words, tiles);
          const Split s = r.split;
          covers("rotary", g, tiles, s);
          CHECK(s.n_chunks <= cap, "rotary: %lld groups, %lld tiles: %d chunks, room for %d", (long long)g, (long long)tiles, s.n_chunks, cap);
          const int64_t slots = r.kernel == RopeKernel::FOUR ? 512 : 256, wgs = g * s.n_chunks;
          CHECK(wgs <= slots || g > slots || wgs > slots + slots / 2, "rotary: %lld groups, %lld tiles: %lld workgroups for %lld slots", (long long)g,
                (long long)tiles, (long long)wgs, (long long)slots);
          // what each kernel's buffers hold
          CHECK(r.kernel != RopeKernel::WAVE || words <= (n_qh <= 4 ? 16 : 8), "wavefront kernel: %d heads, %d words", n_qh, words);
          CHECK(r.kernel != RopeKernel::FOUR || (n_qh > 4 && words <= 16), "four-wavefront kernel: %d heads, %d words", n_qh, words);
        }
    }
  }
  if (bad == 0) std::printf("OK\n");
  return bad ? 1 : 0;
}
