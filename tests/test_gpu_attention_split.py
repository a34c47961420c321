"""Latent attention where its split of the tokens over workgroups changes: one tile, two, the
smallest chunk (8 tiles) and one more, chunks of unequal size, more (sequence, KV head) groups
than workgroups fit at once, one to sixteen query heads per KV head and record widths of every
kernel shape, against the oracle's attention over its fp64 reconstruction of the same records
(stale random words around them). The bar is that of the other attention tests on identical
bytes."""
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
    # key widths, value widths, tokens, batch, KV heads, query heads per KV head
    ([4, 2, 0, 0], [3, 1, 1, 0], 1, 1, 1, 4),
    ([4, 2, 0, 0], [3, 1, 1, 0], 65, 2, 1, 7),
    ([2, 0, 0, 0], [5, 3, 1, 0], 64 * 9, 1, 2, 4),
    ([5, 3, 2, 2], [2, 3, 4, 3], 64 * 10 + 1, 1, 2, 9),
    ([4, 2, 0, 0], [3, 1, 1, 0], 64 * 131 + 7, 1, 8, 4),     # unequal chunks
    ([5, 3, 2, 2], [2, 3, 4, 3], 64 * 70 + 1, 1, 8, 7),      # two workgroups per CU
    ([3, 1, 0, 0], [1, 1, 1, 0], 64 * 40, 1, 1, 16),
    ([8, 6, 4, 2], [8, 8, 3, 1], 64 * 17 + 30, 1, 2, 4),     # wider records
    ([2, 1, 0, 0], [2, 0, 0, 1], 64 * 11 + 5, 300, 3, 1),    # more groups than workgroups fit at once
]


@pytest.mark.parametrize("kw,vw,T,batch,kv,nqh", CASES)
def test_attention_split(kw, vw, T, batch, kv, nqh):
    rng = np.random.default_rng([T, batch, kv, nqh])
    n = min(batch * kv, 12)                            # streams past these repeat them
    ck, pk, cap, kh = make_layer_cache(rng, 128, kw, T, 0, n, g=32)
    cv, pv, _, vh = make_layer_cache(rng, 128, vw, T, 0, n, g=32)
    if n < batch * kv:
        r = batch * kv // n
        ck, cv, pk, pv = _repeat(ck, r), _repeat(cv, r), pk.repeat(r), pv.repeat(r)
    q = rng.standard_normal((batch, kv * nqh, 128)).astype(np.float32) * 0.3
    out = S.spectra_decode_attention(ck, cv, pk, pv, cap, T, torch.from_numpy(q).cuda(), kv).cpu().numpy()
    for b in range(batch) if batch < 8 else (0, 1, batch // 2, batch - 1):
        sl = [(b * kv + h) % n for h in range(kv)]
        want = O.attention_mode_a(q[b].astype(np.float64), np.stack([kh[s] for s in sl]), np.stack([vh[s] for s in sl]))
        for h in range(kv * nqh):
            assert rel_l2(out[b, h], want[h]) <= ATTN_SAME_TOL


def _repeat(c, r):
    out = S.Codec(c.params, c.n_streams * r)
    for name in ("basis", "mean", "bits"):
        getattr(out, name).copy_(torch.cat([getattr(c, name)] * r))
    return out
