"""Per-head reconstruction at the edges of its tiles: every code width 1..8 in every slot, one
to four kept groups, windows around the 64-token tiles, bases far from unit scale, against
the oracle's fp64 decode of the same records (stale random words around them).

The bar is that of the other decode tests (1e-6 relative L2): fp32 sums over at most 128
coefficients of entries split with 2^-22 relative error."""
import numpy as np
import pytest

import paper_2608_07915_amd as S
from gpu_parity import rel_l2
from layer_records import make_layer_cache, repeat_streams

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

CASES = [
    # widths of the four groups, tokens, first slot, streams, basis scale
    ([8, 7, 6, 5], 63, 0, 2, 1.0),
    ([4, 3, 2, 1], 65, 1, 2, 1.0),
    ([1, 2, 3, 4], 129, 63, 1, 2.0 ** 30),
    ([5, 6, 7, 8], 64, 64, 1, 2.0 ** -30),
    ([0, 0, 0, 3], 1, 37, 3, 1.0),
    ([0, 7, 0, 5], 1000, 5, 2, 1.0),
    ([2, 0, 0, 0], 300, 0, 40, 1.0),
    ([0, 0, 0, 0], 70, 2, 1, 1.0),
    ([8, 8, 8, 8], 5000, 31, 1, 1.0),
]


@pytest.mark.parametrize("widths,T,t0,n,scale", CASES)
def test_decode_edges(widths, T, t0, n, scale):
    rng = np.random.default_rng([T, t0, n])
    codec, packed, t_cap, want = make_layer_cache(rng, 128, widths, T, t0, n, scale, g=32)
    got = S.spectra_decode(codec, packed, t_cap, t0, T).cpu().numpy()
    for s in range(n):
        assert rel_l2(got[s], want[s]) <= 1e-6


LONG = [
    # widths, tokens, first slot, streams, times over: 256 CUs of eight wavefronts in all
    ([8, 7, 6, 5], 64 * 130 + 9, 37, 4, 10),   # 48 wavefronts per stream: two or three tiles each
    ([1, 2, 3, 4], 64 * 130 - 3, 0, 4, 10),
    ([0, 5, 0, 3], 64 * 60, 63, 2, 40),        # 24 per stream
    ([3, 2, 1, 0], 64 * 11 + 1, 31, 3, 90),    # one workgroup per stream: one or two tiles
    ([4, 2, 0, 0], 64 * 4, 0, 3, 90),          # half tiles, every wavefront one
    ([2, 0, 1, 0], 64 * 5 - 1, 1, 3, 90),      # five tiles, more than the halves' round
    ([6, 3, 0, 0], 64, 33, 4, 80),             # two tiles: four wavefronts, two workgroups per CU
]


@pytest.mark.parametrize("widths,T,t0,n,times", LONG)
def test_decode_several_tiles_per_wavefront(widths, T, t0, n, times):
    """Wavefronts that walk several tiles (the next tile's words in flight, scales in LDS again)
    and some that walk one fewer, with ragged ends; grids around their limits."""
    rng = np.random.default_rng([T, t0, n])
    codec, packed, t_cap, want = make_layer_cache(rng, 128, widths, T, t0, n, g=32)
    codec, packed = repeat_streams(codec, packed, times)
    got = S.spectra_decode(codec, packed, t_cap, t0, T)
    for s in range(n):
        assert rel_l2(got[s].cpu().numpy(), want[s]) <= 1e-6
        assert torch.equal(got[s::n], got[s].expand(times, T, 128))


def test_decode_infinite_mean():
    """An infinite mean coefficient makes every row of its stream infinite, with the sign of the
    channel's basis entry; other streams stay finite."""
    rng = np.random.default_rng(5)
    codec, packed, t_cap, want = make_layer_cache(rng, 128, [3, 2, 0, 1], 70, 0, 2, g=32)
    codec.mean[0, 40] = float("inf")
    got = S.spectra_decode(codec, packed, t_cap, 0, 70).cpu().numpy()
    sign = np.sign(codec.basis[0, :, 40].cpu().numpy())
    assert np.array_equal(got[0], np.broadcast_to(sign * np.inf, (70, 128)))
    assert rel_l2(got[1], want[1]) <= 1e-6


@pytest.mark.parametrize("weak", [2.0 ** -10, 2.0 ** -17, 2.0 ** -23])
def test_decode_weak_channels(weak):
    """Channels whose basis entries are far smaller than the others' are rebuilt to the same
    relative precision (the bar above holds for them alone: their entries have 22 bits too)."""
    rng = np.random.default_rng(11)
    codec, packed, t_cap, want = make_layer_cache(rng, 128, [4, 2, 0, 1], 300, 0, 2, g=32)
    codec.basis[:, 5:40] *= weak
    got = S.spectra_decode(codec, packed, t_cap, 0, 300).cpu().numpy()
    for s in range(2):
        assert rel_l2(got[s][:, 5:40], want[s][:, 5:40] * weak) <= 1e-6
        assert rel_l2(got[s][:, 40:], want[s][:, 40:]) <= 1e-6
