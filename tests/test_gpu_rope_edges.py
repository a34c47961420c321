"""Rotary attention at the edges of its kernels: every code width 1..8 on both sides, token
counts around the 32-token blocks and 64-token tiles and enough tiles that a wavefront walks
several, one to eight query heads per KV head, record widths on both sides of the dispatch
(8 and 16 words), positions other than the last, against the oracle's rotary attention over
its fp64 reconstruction of the same records (stale random words around them).

The bar is that of the other attention tests on identical bytes (2e-5 relative L2: softmax
weights as two bf16 parts, 2^-17 each)."""
import numpy as np
import pytest

import oracle as O
import paper_2608_07915_amd as S
from gpu_parity import ATTN_SAME_TOL, rel_l2
from layer_records import make_layer_cache

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
    ([5, 3, 2, 2], [2, 3, 4, 3], 4200, 1, 1, 4, None),      # 16-word records, several tiles per wavefront
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
