"""The reduction of the partial sums at the start of a stage's kernel: one wave takes them two by two, 128 at a time, so
that lengths whose launches have odd numbers of blocks, and numbers around 128, 256 and 512, are where it can go wrong."""
import numpy as np
import pytest

from gpu_harness import check_parity, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dist", [0, 1, 2])
@pytest.mark.parametrize("blocks", [19, 127, 128, 129, 257, 511, 512])
def test_any_number_of_partial_sums(oracle, blocks, dist):
    d = (8 * blocks - 3) * 256 - 5  # eight tiles of 256 elements a block, the last block and tile not full
    rng = np.random.default_rng(100 * blocks + dist)
    g = (rng.standard_t(3.0, d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 1e-4, d).astype(np.float32)
    for M in (1, 2, 3):
        ratios = oracle.schedule(0.01, M, 0.25)
        check_parity(oracle, g, r, dist, ratios, run_gpu(g, r, dist, ratios), label=f"{blocks} blocks, law {dist}, M={M}")
