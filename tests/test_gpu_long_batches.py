"""Batches of 60 M elements and more, whose first pass places its blocks piece by piece, behind a call of the same layout:
blocks that moved carry the sums above their tensor's band and the chunks' lists."""
import numpy as np
import pytest

from gpu_harness import batch_plan

pytestmark = pytest.mark.gpu

# a few long tensors, whose partial sums a kernel of its own folds, and many shorter ones; tensors of a few entries between them
FEW = [300, 39_999_973, 1, 20_000_257, 17, 64, 255]
MANY = [1, *[1_250_001 + 7_777 * t for t in range(42)], 3, 300, *[2 + 5 * t for t in range(40)], 4_000_003]


@pytest.mark.parametrize("sizes", [FEW, MANY], ids=["few", "many"])
@pytest.mark.parametrize("kind,dist,delta,base_offset", [("f32", 1, 0.001, 0), ("bf16", 2, 0.002, 3)])
def test_pieces_and_bands(oracle, sizes, kind, dist, delta, base_offset):
    from test_gpu_bands import Workspace
    from test_gpu_batched import check_batched
    from test_gpu_typed import narrow
    offsets = [0, *np.cumsum(sizes).tolist()]
    assert offsets[-1] >= 60_000_000 and batch_plan(sizes)[0] > 0
    rng = np.random.default_rng(len(sizes) + dist)
    r = rng.standard_exponential(offsets[-1], dtype=np.float32)
    r *= np.where(rng.random(offsets[-1], dtype=np.float32) < 0.5, np.float32(-1e-3), np.float32(1e-3))
    pairs = []
    with Workspace(sizes) as ws:
        for call in range(2):
            g = rng.standard_normal(offsets[-1], dtype=np.float32) * np.float32(3e-4)
            given = g
            if kind != "f32":
                given, g = narrow(g, kind)
            results, n = ws.run_batched(given, r, offsets, delta, dist, 2, base_offset=base_offset)
            pairs.append(n)
    check_batched(oracle, g, r, offsets, delta, dist, 2, results, f"{kind} law {dist}")
    assert pairs[1] > pairs[0] + 0.002 * offsets[-1], pairs  # the second call's first pass wrote lists


@pytest.mark.parametrize("dist", [0, 1, 2])
@pytest.mark.parametrize("sizes", [[300, 12_000_007, 9_500_003], [1_750_001] * 12 + [64] * 9], ids=["folded", "unfolded"])
def test_the_first_threshold_does_not_depend_on_the_calls_before(sizes, dist):
    """The first stage's sums are grouped in one way whether or not its first pass left lists: the same bits."""
    from test_gpu_batched import run_batched
    offsets = [0, *np.cumsum(sizes).tolist()]
    rng = np.random.default_rng(5)
    g = rng.standard_normal(offsets[-1], dtype=np.float32) * np.float32(1e-3)
    run_batched(g[:1000], None, [0, 1000], 0.01, 0, 2)  # another layout before
    first = run_batched(g, None, offsets, 0.002, dist, 2)
    again = run_batched(g, None, offsets, 0.002, dist, 2)
    for a, b in zip(first, again):
        np.testing.assert_array_equal(a.stats[0].view(np.uint64), b.stats[0].view(np.uint64))
        assert a.etas[0] == b.etas[0]
