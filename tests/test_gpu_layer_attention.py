"""Per-layer decode-step attention at the edges of its kernels: every code width 1..8 on both
sides, token counts around the 32-token blocks, tiles and chunks, one to sixteen kept
groups, head counts that leave rows of a 16- or 32-head block empty, against the oracle's
attention over its fp64 reconstruction of the same records (stale random words around them).

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
    # d, key widths, value widths, tokens, batch, query heads, square-root split
    (256, [8, 7, 6, 5], [4, 3, 2, 1], 33, 1, 2, False),
    (256, [4, 3, 2, 1], [8, 7, 6, 5], 65, 2, 32, False),
    (384, [1, 0, 0, 0, 0, 0], [0, 0, 0, 0, 0, 3], 1, 2, 3, False),
    (512, [8, 7, 6, 5, 4, 3, 2, 1], [1, 2, 3, 4, 5, 6, 7, 8], 517, 1, 28, True),
    (1024, [5, 3] + [2] * 5 + [1] * 4 + [0] * 5, [3] * 9 + [0] * 7, 260, 1, 32, False),
    (1024, [2] * 16, [3] * 16, 128, 1, 8, True),
    (1024, [4] * 14 + [0] * 2, [6] * 9 + [0] * 7, 2100, 1, 24, False),
    (512, [0] * 8, [2] * 8, 100, 1, 4, False),
    (512, [2] * 8, [0] * 8, 100, 1, 4, False),
]


@pytest.mark.parametrize("d,kw,vw,T,batch,hq,split", CASES)
def test_layer_attention_edges(d, kw, vw, T, batch, hq, split):
    rng = np.random.default_rng([d, T, batch, hq])
    n_kv = d // 128
    ck, pk, cap, kh = make_layer_cache(rng, d, kw, T, 0, batch, split=split)
    cv, pv, _, vh = make_layer_cache(rng, d, vw, T, 0, batch, split=split)
    q = rng.standard_normal((batch, hq, 128)).astype(np.float32) * 0.3
    ws = torch.full((S.spectra_layer_attention_workspace_bytes(ck, batch, hq, T),), 0xFF, dtype=torch.uint8, device="cuda")
    out = S.spectra_layer_decode_attention(ck, cv, pk, pv, cap, T, torch.from_numpy(q).cuda(), n_kv, workspace=ws).cpu().numpy()
    for b in range(batch):
        split_heads = lambda x: x.reshape(T, n_kv, 128).transpose(1, 0, 2)  # noqa: E731
        want = O.attention_mode_a(q[b].astype(np.float64), split_heads(kh[b]), split_heads(vh[b]))
        for h in range(hq):
            assert rel_l2(out[b, h], want[h]) <= ATTN_SAME_TOL


@pytest.mark.parametrize("T,masked", [(700, 521), (700, 700), (300, 40), (2100, 2049)])
def test_layer_attention_minus_infinity_scores(T, masked):
    """Keys whose zero point is -inf score -inf for queries with positive sums: they weigh
    nothing, also where every score of a token range is -inf, and where no token is left the
    output is the mean's row."""
    rng = np.random.default_rng([T, masked])
    d, n_kv = 512, 4
    ck, pk, cap, kh = make_layer_cache(rng, d, [4] + [0] * 7, T, 0, 1)
    cv, pv, _, vh = make_layer_cache(rng, d, [3, 2] + [0] * 6, T, 0, 1)
    at = torch.from_numpy(O.physical_index(0, np.arange(masked), 0, cap, ck.record_words)).cuda()
    pk[at] = (pk[at] & 0xFFFF) | -(0x400 << 16)  # fp16 -inf in the upper half
    q = np.repeat(ck.basis[0, :, :64].sum(1).cpu().numpy().reshape(n_kv, 128), 2, 0) * rng.uniform(0.05, 0.2, (8, 1))
    q = q.astype(np.float32)
    out = S.spectra_layer_decode_attention(ck, cv, pk, pv, cap, T, torch.from_numpy(q[None]).cuda(), n_kv).cpu().numpy()[0]
    if masked == T:
        want = np.repeat((cv.mean[0].double() @ cv.basis[0].double().T).cpu().numpy().reshape(n_kv, 128), 2, 0)
    else:
        split_heads = lambda x: x[masked:].reshape(T - masked, n_kv, 128).transpose(1, 0, 2)  # noqa: E731
        want = O.attention_mode_a(q.astype(np.float64), split_heads(kh[0]), split_heads(vh[0]))
    for h in range(8):
        assert rel_l2(out[h], want[h]) <= ATTN_SAME_TOL


LONG = [
    # d, key widths, value widths, tokens, sequences, times over, query heads, square-root split
    (256, [5, 3, 0, 1], [4, 2, 1, 0], 64 * 9 + 40, 4, 64, 2, False),    # a chunk per sequence, 20 blocks of 32 tokens
    (256, [8, 0, 2, 1], [2, 7, 0, 3], 64 * 40 - 5, 4, 32, 8, True),     # 128 sequences: two chunks of 20 tiles
    (512, [3, 2] + [1] * 6, [6, 0, 5, 0, 1, 1, 0, 2], 64 * 50 + 1, 2, 24, 28, False),  # five chunks of eleven tiles, the last of seven
]


@pytest.mark.parametrize("d,kw,vw,T,n,times,hq,split", LONG)
def test_layer_attention_long_chunks(d, kw, vw, T, n, times, hq, split):
    """So many sequences that a score wavefront walks two or three blocks and a value workgroup
    many tiles, some wavefronts one fewer."""
    rng = np.random.default_rng([d, T, hq])
    n_kv, batch = d // 128, n * times
    ck, pk, cap, kh = make_layer_cache(rng, d, kw, T, 0, n, split=split)
    cv, pv, _, vh = make_layer_cache(rng, d, vw, T, 0, n, split=split)
    ck, pk = repeat_streams(ck, pk, times)
    cv, pv = repeat_streams(cv, pv, times)
    q = rng.standard_normal((batch, hq, 128)).astype(np.float32) * 0.3
    out = S.spectra_layer_decode_attention(ck, cv, pk, pv, cap, T, torch.from_numpy(q).cuda(), n_kv).cpu().numpy()
    split_heads = lambda x: x.reshape(T, n_kv, 128).transpose(1, 0, 2)  # noqa: E731
    for b in (0, 1, batch // 2 + 1, batch - 1):
        want = O.attention_mode_a(q[b].astype(np.float64), split_heads(kh[b % n]), split_heads(vh[b % n]))
        for h in range(hq):
            assert rel_l2(out[b, h], want[h]) <= ATTN_SAME_TOL
