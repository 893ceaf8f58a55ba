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


@pytest.mark.parametrize("d,offset,residual", [(24 * ROW - 1, 0, True), (24 * ROW + 257, 31, True), (25 * ROW - 256, 0, False)])
def test_first_pass_of_top_k(oracle, d, offset, residual):
    from test_gpu_topk import check_topk, run_topk
    rng = np.random.default_rng(d + offset)
    g = rng.standard_normal(d, dtype=np.float32)
    r = rng.standard_normal(d, dtype=np.float32) if residual else None
    k = d // 1000
    for call in range(2):  # the second lists what is above an edge under the first one's k-th magnitude
        out = run_topk(g, r, k, grad_offset=offset, res_offset=offset)
        check_topk(oracle, g, r, k, out, label=f"d={d} offset={offset} ec={residual} call {call}")


@pytest.mark.parametrize("d,offset", [(18 * ROW - 1, 0), (18 * ROW + 257, 31)])
def test_calls_of_one_stage_and_dgc(oracle, d, offset):
    """The first, which reads the vector at its waves' own places again, does not change places; the second does."""
    from test_gpu_dgc import check_dgc, run_dgc
    rng = np.random.default_rng(d + offset)
    g = rng.standard_normal(d, dtype=np.float32)
    r = rng.standard_normal(d, dtype=np.float32)
    out = run_gpu(g, r, 0, [0.001], grad_offset=offset, res_offset=offset)
    check_parity(oracle, g, r, 0, [0.001], out, label=f"d={d} one stage")
    out = run_dgc(g, r, 0.001, 0.01, 3, grad_offset=offset, res_offset=offset)
    check_dgc(oracle, g, r, 0.001, 0.01, 3, out, label=f"d={d} DGC")


@pytest.mark.parametrize("d,offset", [(10 * ROW + 3, 3), (18 * ROW + 257, 31)])
@pytest.mark.parametrize("dist", [0, 1, 2])
def test_the_first_threshold_does_not_depend_on_the_calls_before(d, offset, dist):
    """With bands or without: the same sums, to the last bit."""
    rng = np.random.default_rng(d)
    g = rng.standard_normal(d, dtype=np.float32)
    run_gpu(g[:1000], None, 0, [0.1])  # another shape before
    first, again = (run_gpu(g, None, dist, [0.25, 0.004], grad_offset=offset) for _ in range(2))
    np.testing.assert_array_equal(first.stats[0].view(np.uint64), again.stats[0].view(np.uint64))
    assert first.etas[0] == again.etas[0]
