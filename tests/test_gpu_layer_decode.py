"""Per-layer reconstruction at the edges of its tiles: every code width 1..8, token counts
and windows around the 32-token rows and 256-token ranges, every channel-block count, and
bases far from unit scale, against the oracle's fp64 decode of the same records.

The bar is that of the other decode tests (1e-6 relative L2): the kernel sums in fp32
(2^-24 per addition, up to 16 groups) over basis entries split with 2^-22 relative error."""
import numpy as np
import pytest

import oracle as O
import paper_2608_07915_amd as S
from gpu_parity import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

CASES = [
    # d, widths of the groups, tokens, first slot, streams, basis scale, square-root split
    (256, [8, 7, 6, 5], 33, 0, 1, 1.0, False),
    (256, [0, 0, 0, 1], 1, 63, 2, 1.0, False),
    (384, [5, 0, 3, 0, 2, 1], 255, 31, 2, 1.0, True),
    (512, [8, 7, 6, 5, 4, 3, 2, 1], 257, 1, 1, 2.0 ** 30, False),
    (512, [1] * 8, 513, 64, 1, 2.0 ** -30, True),
    (1024, [8] * 7 + [0] * 9, 300, 5, 1, 1.0, False),
    (1024, [2] * 16, 32, 0, 1, 1.0, True),
    (1024, [0] * 16, 70, 0, 1, 1.0, False),
]


@pytest.mark.parametrize("d,widths,T,t0,n,scale,split", CASES)
def test_layer_decode_edges(d, widths, T, t0, n, scale, split):
    rng = np.random.default_rng([d, T, t0, n])
    used = sum(1 + 2 * b for b in widths if b)
    p = O.Params(head_dim=d, group_size=64, ratio=8.0, budget_bits=32 * max(used + 1, 4))
    W, t_cap = O.record_words(p), (t0 + T + 63) // 64 * 64 + 64
    codec = S.Codec(S.Params(head_dim=d, group_size=64, ratio=8.0, budget_bits=p.budget_bits), n, latent_scale=split)
    words = rng.integers(0, 2 ** 32, size=n * t_cap * W, dtype=np.uint32)
    want = []
    for s in range(n):
        q, _ = np.linalg.qr(rng.standard_normal((d, d)))
        basis = (q * scale).astype(np.float32)
        mean = rng.standard_normal(d).astype(np.float32)
        f = np.exp(rng.uniform(-1, 3, d)).astype(np.float32) if split else None
        bits = list(rng.permutation(widths)) if s else widths
        codes = np.zeros((T, d), np.uint8)
        meta = np.zeros((T, d // 64), np.uint32)
        for G, b in enumerate(bits):
            if b:
                codes[:, 64 * G:64 * G + 64] = rng.integers(0, 1 << b, size=(T, 64))
                meta[:, G] = O.codec.fp16_bits(rng.uniform(0, 2, T).astype(np.float16)) | \
                    (O.codec.fp16_bits((-rng.uniform(0, 4, T)).astype(np.float16)) << np.uint32(16))
        rec = O.pack(codes, meta, bits, p)
        for w in range(W):
            words[O.physical_index(s, t0 + np.arange(T), w, t_cap, W)] = rec[:, w]
        codec.basis[s].copy_(torch.from_numpy(basis))
        codec.mean[s].copy_(torch.from_numpy(mean))
        codec.bits[s].copy_(torch.from_numpy(np.asarray(bits, np.uint8)))
        if split:
            codec.lscale[s].copy_(torch.from_numpy(f))
        want.append(O.decode(rec, basis, mean, bits, p, f))
    packed = torch.from_numpy(words.view(np.int32)).cuda()
    got = S.spectra_decode(codec, packed, t_cap, t0, T).cpu().numpy()
    for s in range(n):
        assert rel_l2(got[s], want[s]) <= 1e-6
