"""Codecs and packed records made by hand (random orthogonal basis, given group
widths, random codes and metadata), packed by the oracle, for tests at kernel edges."""
import numpy as np

import oracle as O
import paper_2608_07915_amd as S


def make_layer_cache(rng, d, widths, T, t0, n, scale=1.0, split=False, stale=True, g=64):
    """n streams of T tokens from slot t0 on: (codec, packed, t_capacity, oracle rows [n][T, d]).
    Streams after the first take the widths in another order; slots outside the tokens hold
    random words (`stale`) or zeros. g: group size (64 per layer, 32 per head)."""
    import torch
    used = sum(1 + g // 32 * b for b in widths if b)
    p = O.Params(head_dim=d, group_size=g, ratio=8.0, budget_bits=32 * max(used + 1, 4))
    W, t_cap = O.record_words(p), (t0 + T + 63) // 64 * 64 + 64
    codec = S.Codec(S.Params(head_dim=d, group_size=g, ratio=8.0, budget_bits=p.budget_bits), n, latent_scale=split)
    words = rng.integers(0, 2 ** 32 if stale else 1, size=n * t_cap * W, dtype=np.uint32)
    rows = []
    for s in range(n):
        q, _ = np.linalg.qr(rng.standard_normal((d, d)))
        basis = (q * scale).astype(np.float32)
        mean = rng.standard_normal(d).astype(np.float32)
        f = np.exp(rng.uniform(-1, 3, d)).astype(np.float32) if split else None
        bits = list(rng.permutation(widths)) if s else widths
        codes = np.zeros((T, d), np.uint8)
        meta = np.zeros((T, d // g), np.uint32)
        for G, b in enumerate(bits):
            if b:
                codes[:, g * G:g * G + g] = rng.integers(0, 1 << b, size=(T, g))
                meta[:, G] = O.codec.fp16_bits((rng.uniform(0, 4, T) / 2.0 ** b).astype(np.float16)) | \
                    (O.codec.fp16_bits((-rng.uniform(0, 4, T)).astype(np.float16)) << np.uint32(16))
        rec = O.pack(codes, meta, bits, p)
        for w in range(W):
            words[O.physical_index(s, t0 + np.arange(T), w, t_cap, W)] = rec[:, w]
        codec.basis[s].copy_(torch.from_numpy(basis))
        codec.mean[s].copy_(torch.from_numpy(mean))
        codec.bits[s].copy_(torch.from_numpy(np.asarray(bits, np.uint8)))
        if split:
            codec.lscale[s].copy_(torch.from_numpy(f))
        rows.append(O.decode(rec, basis, mean, bits, p, f))
    return codec, torch.from_numpy(words.view(np.int32)).cuda(), t_cap, rows


def repeat_streams(codec, packed, r):
    """The codec and records with all streams r times over."""
    import torch
    out = S.Codec(codec.params, codec.n_streams * r, latent_scale=codec.lscale is not None)
    for name in ("basis", "mean", "bits") + (("lscale",) if codec.lscale is not None else ()):
        getattr(out, name).copy_(torch.cat([getattr(codec, name)] * r))
    return out, packed.repeat(r)
