"""Rotary attention at the edges of its kernels: every code width 1..8 on both sides, token
counts around the 32-token blocks and 64-token tiles, chunks of one step and of several, one
to eight query heads per KV head, record widths on both sides of the dispatch (8 and 16
words), positions other than the last, against the oracle's rotary attention over its fp64
reconstruction of the same records (stale random words around them).

The bar is that of the other attention tests on identical bytes (1e-5 relative L2: softmax
weights as two bf16 parts, 2^-17 each)."""
import numpy as np
import pytest

import oracle as O
import paper_2608_07915_amd as S
from gpu_parity import ATTN_SAME_TOL, rel_l2
from layer_records import make_layer_cache, repeat_streams

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

CASES = [
    # key widths, value widths, tokens, batch, KV heads, query heads per KV head, position
    ([4, 2, 0, 0], [3, 1, 1, 0], 33, 1, 2, 4, None),
    ([0, 0, 7, 0], [0, 6, 0, 0], 1, 2, 1, 1, 5),
    ([1, 0, 0, 0], [0, 0, 0, 0], 64, 1, 1, 3, None),
    ([0, 0, 0, 0], [5, 0, 0, 1], 65, 1, 1, 4, 1000),
    ([5, 3, 2, 2], [2, 3, 4, 3], 4200, 1, 1, 4, None),      # 16-word records, a last chunk of two tiles
    ([8, 0, 0, 4], [1, 1, 1, 1], 129, 1, 2, 2, 100000),
    ([3, 1, 1, 0], [4, 2, 0, 0], 2300, 1, 1, 7, None),      # eight heads at 8 words
    ([6, 1, 0, 0], [1, 2, 1, 0], 31, 2, 1, 8, None),
    ([7, 5, 0, 0], [3, 3, 3, 2], 200, 1, 2, 6, None),       # five to eight heads, 9 to 16 words
    ([8, 6, 4, 2], [8, 8, 3, 1], 130, 1, 1, 4, None),       # wider records
]


@pytest.mark.parametrize("kw,vw,T,batch,kv,nqh,pos", CASES)
def test_rope_attention_edges(kw, vw, T, batch, kv, nqh, pos):
    rng = np.random.default_rng([T, batch, kv, nqh])
    ck, pk, cap, kh = make_layer_cache(rng, 128, kw, T, 0, batch * kv, g=32)
    cv, pv, _, vh = make_layer_cache(rng, 128, vw, T, 0, batch * kv, g=32)
    q = rng.standard_normal((batch, kv * nqh, 128)).astype(np.float32) * 0.3
    w = (1.0e4 ** (-np.arange(64) / 64)).astype(np.float32)
    out = S.spectra_decode_attention_rope(ck, cv, pk, pv, cap, T, torch.from_numpy(q).cuda(), kv,
                                          torch.from_numpy(w).cuda(), q_position=pos).cpu().numpy()
    for b in range(batch):
        sl = slice(b * kv, (b + 1) * kv)
        want = O.attention_mode_a_rope(q[b].astype(np.float64), np.stack(kh[sl]), np.stack(vh[sl]), w.astype(np.float64),
                                       T - 1 if pos is None else pos)
        for h in range(kv * nqh):
            assert rel_l2(out[b, h], want[h]) <= ATTN_SAME_TOL


LONG = [
    # key widths, value widths, tiles, query heads per KV head: 128 (sequence, KV head) groups, so
    # chunks are half of the tiles
    ([4, 2, 0, 0], [3, 1, 1, 0], 40, 4),     # a tile per wavefront: two or three tiles each
    ([5, 3, 2, 2], [2, 3, 4, 3], 40, 3),     # the same with 16-word records
    ([3, 1, 1, 0], [4, 2, 0, 0], 40, 7),     # eight heads
    ([3, 1, 1, 0], [4, 2, 0, 0], 19, 7),     # chunks of ten tiles: four wavefronts per tile
    ([7, 5, 0, 0], [3, 3, 3, 2], 40, 6),     # 16 words, five to eight heads
    ([8, 6, 4, 2], [8, 8, 3, 1], 12, 4),     # wider records
]


@pytest.mark.parametrize("kw,vw,tiles,nqh", LONG)
def test_rope_attention_long_chunks(kw, vw, tiles, nqh):
    """Chunks of several steps of every kernel: the turn from one tile to the next, words
    loaded ahead, buffers used again, sums rescaled."""
    rng = np.random.default_rng([tiles, nqh])
    batch, kv, n, T = 64, 2, 8, 64 * tiles - 23
    ck, pk, cap, kh = make_layer_cache(rng, 128, kw, T, 0, n, g=32)
    cv, pv, _, vh = make_layer_cache(rng, 128, vw, T, 0, n, g=32)
    ck, pk = repeat_streams(ck, pk, batch * kv // n)
    cv, pv = repeat_streams(cv, pv, batch * kv // n)
    q = rng.standard_normal((batch, kv * nqh, 128)).astype(np.float32)
    q *= np.exp(rng.uniform(-2, 1, (batch, kv * nqh, 1))).astype(np.float32)
    w = (1.0e4 ** (-np.arange(64) / 64)).astype(np.float32)
    out = S.spectra_decode_attention_rope(ck, cv, pk, pv, cap, T, torch.from_numpy(q).cuda(), kv,
                                          torch.from_numpy(w).cuda()).cpu().numpy()
    for b in (0, 1, 33, 63):
        sl = [(b * kv + h) % n for h in range(kv)]
        want = O.attention_mode_a_rope(q[b].astype(np.float64), np.stack([kh[s] for s in sl]), np.stack([vh[s] for s in sl]),
                                       w.astype(np.float64), T - 1)
        for h in range(kv * nqh):
            assert rel_l2(out[b, h], want[h]) <= ATTN_SAME_TOL
