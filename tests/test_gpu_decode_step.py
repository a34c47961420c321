"""spectra_decode_step (append the new key/value, then attend) against the two
separate calls it replaces: spectra_encode of the new token into slot t, then
spectra_decode_attention over t + 1 tokens. Records must be byte-identical and
outputs identical; both are checked against the oracle by the encode and
attention parity tests."""
import numpy as np
import pytest

import oracle as O
import paper_2608_07915_amd as S
import synth
from gpu_parity import fit_and_encode, to_device
from layer_records import make_layer_cache, repeat_streams

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def _streams(w, T, batch, tensor):
    return np.stack([synth.numpy_stream(w, b, 0, h, tensor, n_tokens=T) for b in range(batch)
                     for h in range(w.n_kv_heads)])


@pytest.mark.parametrize("name,T0,batch,ratio,kappa", [("llama_layer_4x", 61, 2, 8.0, 0.5), ("tiny", 127, 1, 8.0, 0.5),
                                                       ("qwen_layer_8x", 700, 1, 12.0, 0.5),
                                                       ("llama_layer_4x", 500, 1, 16 / 9, 0.5),
                                                       ("llama_layer_4x", 61, 1, 8.0, 0.25),
                                                       ("qwen_layer_8x", 190, 1, 4.0, 0.7)])
def test_decode_step_equals_encode_then_attention(name, T0, batch, ratio, kappa):
    """kappa != 1/2: key and value records of different widths (asymmetric split)."""
    w = synth.WORKLOADS[name]
    n_steps = 5                                   # crosses a 64-token tile boundary for T0 = 61 / 127
    T = T0 + n_steps
    t_cap = (T + 63) // 64 * 64
    xk, xv = _streams(w, T, batch, 0), _streams(w, T, batch, 1)
    dk, dv = to_device(xk, w.dtype), to_device(xv, w.dtype)
    p_k = p_v = O.Params(ratio=ratio)
    if kappa != 0.5:
        p_k, p_v = O.split_budget(p_k, kappa)
    ck, pk = fit_and_encode(dk[:, :T0].contiguous(), p_k, t_cap)
    cv, pv = fit_and_encode(dv[:, :T0].contiguous(), p_v, t_cap)
    pk2, pv2 = pk.clone(), pv.clone()
    H, Hq = w.n_kv_heads, w.n_q_heads
    for i in range(n_steps):
        t = T0 + i
        q = to_device(np.stack([synth.numpy_query(w, b, 0, i) for b in range(batch)]), w.dtype)
        # separate calls
        S.spectra_encode(ck, dk[:, t:t + 1], t, pk, t_cap)
        S.spectra_encode(cv, dv[:, t:t + 1], t, pv, t_cap)
        want = S.spectra_decode_attention(ck, cv, pk, pv, t_cap, t + 1, q, H)
        # fused
        k_new = dk[:, t].reshape(batch, H, 128).contiguous()
        v_new = dv[:, t].reshape(batch, H, 128).contiguous()
        got = S.spectra_decode_step(ck, cv, pk2, pv2, t_cap, t, k_new, v_new, q, H)
        torch.cuda.synchronize()
        assert torch.equal(pk, pk2), (name, t)
        assert torch.equal(pv, pv2), (name, t)
        assert torch.equal(got, want), (name, t)
        assert got.shape == (batch, Hq, 128)


@pytest.mark.parametrize("T0,batch,kv,nqh,widths", [
    # where the append, the workspace or a queue could move the cuts between workgroups
    (19999, 1, 8, 4, ([4, 2, 0, 0], [3, 1, 1, 0])),
    (30000, 1, 8, 4, ([2, 1, 0, 0], [2, 0, 0, 1])),
    (29999, 1, 8, 4, ([5, 3, 2, 2], [2, 3, 4, 3])),
    (33000, 1, 4, 7, ([4, 2, 0, 0], [3, 1, 1, 0])),
    (11999, 5, 8, 4, ([5, 3, 2, 2], [2, 3, 4, 3])),
    (4000, 5, 8, 4, ([4, 2, 0, 0], [3, 1, 1, 0])),
    (999, 16, 8, 4, ([4, 2, 0, 0], [3, 1, 1, 0])),
])
def test_decode_step_long_caches(T0, batch, kv, nqh, widths):
    """The same over caches of many chunks, with the smallest workspace and a larger one: the sums
    are split alike, so the outputs are identical."""
    rng = np.random.default_rng([T0, batch, kv])
    n, t_cap = batch * kv, (T0 + 64) // 64 * 64
    g = torch.Generator(device="cuda").manual_seed(T0)
    caches = []
    for w in widths:
        codec, packed, _, _ = make_layer_cache(rng, 128, w, 64, 0, 4, g=32)
        codec, _ = repeat_streams(codec, packed, n // 4)
        x = torch.randn((n, T0 + 1, 128), generator=g, device="cuda", dtype=torch.bfloat16)
        rec = codec.empty_packed(t_cap)
        S.spectra_encode(codec, x[:, :T0].contiguous(), 0, rec, t_cap)
        caches.append((codec, rec, x[:, T0].reshape(batch, kv, 128).contiguous()))
    (ck, pk, k_new), (cv, pv, v_new) = caches
    q = 0.3 * torch.randn((batch, kv * nqh, 128), generator=g, device="cuda")
    need = S.spectra_attention_workspace_bytes(batch, kv * nqh, kv, T0 + 1)
    got = [S.spectra_decode_step(ck, cv, pk, pv, t_cap, T0, k_new, v_new, q, kv,
                                 workspace=torch.empty(r * need, dtype=torch.uint8, device="cuda")) for r in (1, 4)]
    want = [S.spectra_decode_attention(ck, cv, pk, pv, t_cap, T0 + 1, q, kv,
                                       workspace=torch.empty(r * need, dtype=torch.uint8, device="cuda")) for r in (1, 4)]
    assert torch.isfinite(want[0]).all()
    for o in got + want[1:]:
        assert torch.equal(o, want[0]), (T0, batch)
