"""Per-layer reconstruction at the edges of its tiles: every code width 1..8, token counts
and windows around the 32-token rows and 256-token ranges, every channel-block count, and
bases far from unit scale, against the oracle's fp64 decode of the same records.

The bar is that of the other decode tests (1e-6 relative L2): the kernel sums in fp32
(2^-24 per addition, up to 16 groups) over basis entries split with 2^-22 relative error."""
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
    codec, packed, t_cap, want = make_layer_cache(rng, d, widths, T, t0, n, scale, split)
    got = S.spectra_decode(codec, packed, t_cap, t0, T).cpu().numpy()
    for s in range(n):
        assert rel_l2(got[s], want[s]) <= 1e-6


@pytest.mark.parametrize("weak", [2.0 ** -10, 2.0 ** -17, 2.0 ** -23])
@pytest.mark.parametrize("split", [False, True])
def test_layer_decode_weak_channels(split, weak):
    """Channels whose basis entries are far smaller than the others' are rebuilt to the same
    relative precision (the bar above holds for them alone: their entries have 22 bits too)."""
    rng = np.random.default_rng(11)
    codec, packed, t_cap, want = make_layer_cache(rng, 512, [4, 2, 1, 0, 3, 0, 0, 1], 300, 0, 2, split=split)
    codec.basis[:, 5:40] *= weak
    got = S.spectra_decode(codec, packed, t_cap, 0, 300).cpu().numpy()
    for s in range(2):
        assert rel_l2(got[s][:, 5:40], want[s][:, 5:40] * weak) <= 1e-6
        assert rel_l2(got[s][:, 40:], want[s][:, 40:]) <= 1e-6


LONG = [
    # d, widths, tokens, first slot, streams, times over, square-root split
    (256, [5, 3, 0, 8], 256 * 5 + 70, 17, 4, 32, True),             # one workgroup per block: six ranges each
    (384, [4, 0, 3, 1, 7, 2], 256 * 9 - 1, 0, 2, 14, True),         # three per block: three ranges each
    (1024, [2] * 12 + [0] * 4, 256 * 7 + 1, 64, 1, 8, False),       # four per block: two ranges each
]


@pytest.mark.parametrize("d,widths,T,t0,n,times,split", LONG)
def test_layer_decode_several_ranges(d, widths, T, t0, n, times, split):
    """So many streams that a workgroup walks several ranges with the same staged blocks."""
    rng = np.random.default_rng([d, T, t0])
    codec, packed, t_cap, want = make_layer_cache(rng, d, widths, T, t0, n, split=split)
    codec, packed = repeat_streams(codec, packed, times)
    got = S.spectra_decode(codec, packed, t_cap, t0, T)
    for s in range(n):
        assert rel_l2(got[s].cpu().numpy(), want[s]) <= 1e-6
        assert torch.equal(got[s::n], got[s].expand(times, T, d))
