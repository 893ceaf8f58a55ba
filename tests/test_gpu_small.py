"""Vectors that one block handles: the ends of its rows of float4s, the last incomplete float4, the longest vector of either
shape, and first thresholds that nearly everything exceeds, so that a wave's list is too short and it goes on without."""
import numpy as np
import pytest

from gpu_harness import check_parity, run_gpu

pytestmark = pytest.mark.gpu

# a row is 960 float4s; 4 rows are the shorter shape, 10 (of which 36,864 elements fill 9.6) the longer one
LENGTHS = [1, 2, 3, 4, 5, 3839, 3840, 3841, 11521, 15359, 15360, 15361, 15363, 34561, 36863, 36864]


@pytest.mark.parametrize("dist", [0, 1, 2])
@pytest.mark.parametrize("ec", [True, False])
def test_ends_of_rows(oracle, dist, ec):
    for d in LENGTHS:
        rng = np.random.default_rng(10 * d + dist)
        g = (rng.standard_t(3.0, d) * 1e-3).astype(np.float32)
        r = rng.laplace(0, 1e-3, d).astype(np.float32) if ec else None
        for M in (1, 3):
            ratios = oracle.schedule(0.01, M, 0.25)
            out = run_gpu(g, r, dist, ratios, grad_offset=d % 4, res_offset=d % 3)
            check_parity(oracle, g, r, dist, ratios, out, label=f"d={d} law {dist} M={M} ec={ec}")


@pytest.mark.parametrize("dist", [0, 1, 2])
@pytest.mark.parametrize("d", [9000, 20011, 36864])
@pytest.mark.parametrize("ratios", [(0.97,), (0.97, 0.9), (0.6, 0.9, 0.9, 0.5), (0.45, 0.5, 0.02)])
def test_lists_that_are_too_short(oracle, d, dist, ratios):
    rng = np.random.default_rng(d + dist)
    g = rng.laplace(0, 1e-3, d).astype(np.float32)
    r = rng.laplace(0, 1e-3, d).astype(np.float32)
    for cap in (None, d // 7):  # the second: the output is full long before the end
        out = run_gpu(g, r, dist, ratios, cap=cap)
        check_parity(oracle, g, r, dist, ratios, out, capacity=cap, label=f"d={d} law {dist} ratios {ratios} cap {cap}")


@pytest.mark.parametrize("kind", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("d", [3839, 3841, 15359, 15361, 26_001, 36_863])
def test_mild_ratios(oracle, kind, d):
    """One stage with and without lists (the line is 0.15) for each number of rows, the types that share a kernel, and calls with
    and without a residual, which do."""
    import paper_2101_10761_amd as sidco
    from test_gpu_typed import narrow, run_typed
    rng = np.random.default_rng(3 * d)
    g = (rng.standard_t(3.0, d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 1e-3, d).astype(np.float32)
    for dist in (0, 1, 2):
        for delta, stages in ((0.14, 1), (0.16, 1), (0.6, 1), (0.1, 2)):
            ratios = sidco.sidco_stage_ratios(delta, stages)
            for res in (r, None):
                label = f"{kind} d={d} law {dist} delta {delta} M={stages} ec={res is not None}"
                if kind == "f32":
                    cap = None
                    out, seen = run_gpu(g, res, dist, ratios, grad_offset=1, res_offset=2), g
                else:
                    cap = sidco.sidco_out_capacity(d, delta)
                    given, seen = narrow(g, kind)
                    out = run_typed(given, res, dist, delta, stages, grad_offset=1, res_offset=2)
                check_parity(oracle, seen, res, dist, ratios, out, capacity=cap, label=label)
