"""The first pass's tiles where the waves begin to change places from row to row: whole rows, one tile more or less, an
incomplete last tile and an incomplete first one (a vector that starts inside a line), without and with bands."""
import numpy as np
import pytest

from gpu_harness import check_parity, run_gpu

pytestmark = pytest.mark.gpu

ROW = 4096 * 256  # elements of a row of tiles


@pytest.mark.parametrize("d,offset,residual", [(18 * ROW - 1, 0, True), (18 * ROW, 0, True), (18 * ROW, 5, True), (18 * ROW + 257, 31, True),
                                               (19 * ROW - 256, 0, False), (19 * ROW + 2048 * 256 + 2, 1, True)])
def test_first_pass_on_both_sides_of_the_line(oracle, d, offset, residual):
    rng = np.random.default_rng(d + offset)
    g = rng.standard_normal(d, dtype=np.float32)
    r = rng.standard_normal(d, dtype=np.float32) if residual else None
    ratios = oracle.schedule(0.001, 2, 0.25)
    for call in range(2):  # the second goes by the first one's thresholds
        out = run_gpu(g, r, 0, ratios, grad_offset=offset, res_offset=offset)
        check_parity(oracle, g, r, 0, ratios, out, label=f"d={d} offset={offset} ec={residual} call {call}")
