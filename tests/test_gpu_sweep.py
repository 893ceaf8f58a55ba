"""GPU parity where the split of the vector into waves' tiles changes shape: fewer tiles than waves, a tile more or less
than a whole round of 4096 waves, an incomplete last tile owned by a middle or the last wave, one tile (in a batch); and
on both sides of the lengths and ratios where a call takes other kernels.  Single vectors of up to ONE_BLOCK elements
have no tiles: one block takes them as a whole."""
import numpy as np
import pytest

from gpu_harness import batch_plan, check_parity, run_gpu

pytestmark = pytest.mark.gpu

ROUND = 4096 * 256  # elements of one tile for every wave


@pytest.mark.parametrize("d", [1, 255, 256, 257, 8 * 256 + 1, ROUND - 256, ROUND - 1, ROUND, ROUND + 1, ROUND + 257,
                               2 * ROUND + 100, 3 * ROUND - 255])
@pytest.mark.parametrize("dist,delta,stages", [(0, 0.02, 1), (2, 0.01, 3), (1, 0.002, 2)])
def test_edges_of_the_tile_split(oracle, d, dist, delta, stages):
    rng = np.random.default_rng(d + dist)
    ratios = oracle.schedule(delta, stages, 0.25)
    g = (rng.standard_t(3.0, size=d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=d).astype(np.float32)
    for residual in (r, None):
        out = run_gpu(g, residual, dist, ratios)
        check_parity(oracle, g, residual, dist, ratios, out, label=f"d={d} dist={dist} M={stages} ec={residual is not None}")


@pytest.mark.parametrize("d", [ROUND + 257, 2 * ROUND - 1])
@pytest.mark.parametrize("stages", [2, 3])
def test_dense_fallback_walks_the_same_tiles(oracle, d, stages):
    """Candidate lists that start above the next threshold: the stages behind the dense one read the vector again."""
    import paper_2101_10761_amd as sidco
    rng = np.random.default_rng(d + stages)
    g = rng.uniform(-1e-3, 1e-3, size=d).astype(np.float32)   # far lighter tail than the fitted law
    ratios = oracle.schedule(0.001, stages, 0.25)
    sidco.sidco_set_speculation(1.0)
    try:
        out = run_gpu(g, None, 0, ratios)
    finally:
        sidco.sidco_set_speculation(0.5)
    assert out.status & sidco.ST_FALLBACK
    check_parity(oracle, g, None, 0, ratios, out, label=f"fallback d={d} M={stages}")


@pytest.mark.parametrize("n_short,n_long", [(500, 12), (400, 112), (0, 512), (511, 1), (3, 1)])
def test_batch_of_more_blocks_than_one_vector_uses(oracle, n_short, n_long):
    """Many short vectors beside long ones: the short ones' blocks come on top of the long ones' 512."""
    from test_gpu_batched import check_batched, run_batched
    rng = np.random.default_rng(n_short + 3 * n_long)
    sizes = np.concatenate([rng.integers(1, 700, n_short), rng.integers(9_000, 60_000 if n_long > 12 else 400_000, n_long)])
    rng.shuffle(sizes)
    offs = [0] + [int(v) for v in np.cumsum(sizes)]
    g = (rng.standard_t(3.0, size=offs[-1]) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=offs[-1]).astype(np.float32)
    for dist, delta, stages in ((2, 0.01, 3), (0, 0.02, 1)):
        out = run_batched(g, r, offs, delta, dist, stages, repeat=2)
        check_batched(oracle, g, r, offs, delta, dist, stages, out, f"{n_short} short, {n_long} long, M={stages}")


@pytest.mark.parametrize("d", [1, 2, 3, 5, 254, 255, 256, 257, 511, ROUND - 2, ROUND + 255, 12_000_001])
@pytest.mark.parametrize("grad_offset,res_offset", [(1, 1), (3, 3), (2, 0), (0, 3), (1, 2)])
def test_buffers_off_the_16_byte_grid(oracle, d, grad_offset, res_offset):
    """Tiles follow the alignment of the accumulated vector; the gradient may have another one."""
    rng = np.random.default_rng(d + 10 * grad_offset + res_offset)
    g = (rng.standard_t(3.0, size=d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=d).astype(np.float32)
    for residual, dist, stages in ((r, 2, 3), (None, 0, 1)):
        if d > ROUND + 255 and residual is None:
            continue
        ratios = oracle.schedule(0.01, stages, 0.25)
        out = run_gpu(g, residual, dist, ratios, grad_offset=grad_offset, res_offset=res_offset)
        check_parity(oracle, g, residual, dist, ratios, out, label=f"d={d} offsets {grad_offset},{res_offset} M={stages}")


@pytest.mark.parametrize("dtype", ["bfloat16", "float16"])
@pytest.mark.parametrize("base", [1, 2, 3, 6])
@pytest.mark.parametrize("ec", [True, False])
def test_16_bit_batches_off_the_grid(oracle, dtype, base, ec):
    import torch
    from test_gpu_batched import check_batched, run_batched
    rng = np.random.default_rng(base)
    offs = [0] + [int(v) for v in np.cumsum(rng.integers(1, 3000, 40))] + [150_001]
    g16 = torch.from_numpy((rng.standard_t(3.0, size=offs[-1]) * 1e-2).astype(np.float32)).to(getattr(torch, dtype))
    g = g16.to(torch.float32).numpy()
    r = rng.laplace(0, 3e-3, size=offs[-1]).astype(np.float32) if ec else None
    out = run_batched(g16, r, offs, 0.02, 2, 2, base_offset=base, repeat=2)
    check_batched(oracle, g, r, offs, 0.02, 2, 2, out, f"{dtype} base {base} ec={ec}")


def test_16_bit_batch_without_residual_may_start_inside_its_buffer(oracle):
    """offsets[0] > 0: the widened copy of the tensors starts at the first tensor, not at the buffer's element 0."""
    import torch
    from test_gpu_batched import check_batched, run_batched
    rng = np.random.default_rng(5)
    start, sizes = 3_000_000, [70_001, 5, 20_000]
    offs = [start] + [start + int(v) for v in np.cumsum(sizes)]
    full = (rng.standard_t(3.0, size=offs[-1]) * 1e-2).astype(np.float32)
    g16 = torch.from_numpy(full).to(torch.bfloat16)
    import paper_2101_10761_amd as sidco
    need = sidco.sidco_workspace_bytes_batched_typed(offs, sidco.GRAD_BF16, False)
    ws = torch.full((need + 16_000_000,), 0x5a, dtype=torch.uint8, device="cuda:0")   # slack that nothing may touch
    sidco.sidco_set_workspace(ws[:need])
    try:
        out = run_batched(g16, None, offs, 0.02, 2, 2)
    finally:
        sidco.sidco_set_workspace(None)
    assert torch.all(ws[need:] == 0x5a)
    check_batched(oracle, g16.to(torch.float32).numpy(), None, offs, 0.02, 2, 2, out, "start inside the buffer")


@pytest.mark.parametrize("d", [1, 31, 225, 226, 256, 287, 481, ROUND - 16])
@pytest.mark.parametrize("grad_offset,res_offset", [(5, 5), (16, 16), (31, 31), (0, 30), (29, 4)])
def test_buffers_off_the_line_grid(oracle, d, grad_offset, res_offset):
    """Tiles sit on the 128-byte lines of the accumulated vector (a whole round less a tile's end; the short lengths, one
    block each, go through unaligned accesses there)."""
    rng = np.random.default_rng(d + 100 * grad_offset + res_offset)
    g = (rng.standard_t(3.0, size=d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=d).astype(np.float32)
    for residual, dist, stages in ((r, 2, 3), (None, 0, 1)):
        ratios = oracle.schedule(0.01, stages, 0.25)
        out = run_gpu(g, residual, dist, ratios, grad_offset=grad_offset, res_offset=res_offset)
        check_parity(oracle, g, residual, dist, ratios, out, label=f"d={d} offsets {grad_offset},{res_offset} M={stages}")


def test_batch_of_tensors_that_end_inside_lines(oracle):
    """Tensors at every place inside a 128-byte line, of one tile and of two tiles that are both incomplete."""
    from test_gpu_batched import check_batched, run_batched
    rng = np.random.default_rng(3)
    sizes = [n for k in range(34) for n in (225 + k, 1 + k, 481 + k)]
    offs = [0] + [int(v) for v in np.cumsum(sizes)]
    g = (rng.standard_t(3.0, size=offs[-1]) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=offs[-1]).astype(np.float32)
    for residual, dist, delta, stages in ((r, 2, 0.01, 3), (None, 0, 0.02, 1)):
        out = run_batched(g, residual, offs, delta, dist, stages, repeat=2)
        check_batched(oracle, g, residual, offs, delta, dist, stages, out, f"ends inside lines M={stages}")


ONE_BLOCK = 36_864  # the longest vector that one block takes as a whole


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 63, 4095, 4097, 12_287, 12_288, 12_289, ONE_BLOCK - 1, ONE_BLOCK, ONE_BLOCK + 1])
@pytest.mark.parametrize("dist,delta,stages", [(0, 0.02, 1), (2, 0.01, 3), (1, 0.002, 2), (0, 0.001, 8)])
def test_one_block_calls(oracle, d, dist, delta, stages):
    rng = np.random.default_rng(d + dist + stages)
    ratios = oracle.schedule(delta, stages, 0.25)
    g = (rng.standard_t(3.0, size=d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=d).astype(np.float32)
    for residual, cap, offs in ((r, None, (0, 0)), (None, None, (1, 0)), (r, max(1, d // 200), (3, 1))):
        out = run_gpu(g, residual, dist, ratios, cap=cap, grad_offset=offs[0], res_offset=offs[1])
        check_parity(oracle, g, residual, dist, ratios, out, capacity=cap, label=f"d={d} dist={dist} M={stages} cap={cap} {offs}")
        if stages == 1 and d <= ONE_BLOCK:
            again = run_gpu(g, residual, dist, ratios, cap=cap, grad_offset=offs[0], res_offset=offs[1])
            np.testing.assert_array_equal(again.idx, out.idx)  # a single stage's order is fixed


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("d", [1, 3, 12_289, ONE_BLOCK - 2, ONE_BLOCK + 1])
def test_one_block_calls_on_16_bit_gradients(oracle, kind, d):
    from test_gpu_typed import narrow, run_typed
    rng = np.random.default_rng(d)
    g16, g = narrow((rng.standard_t(3.0, size=d) * 1e-2).astype(np.float32), kind)
    r = rng.laplace(0, 3e-3, size=d).astype(np.float32)
    for residual in (r, None):
        out = run_typed(g16, residual, 2, 0.01, 2, grad_offset=1, res_offset=1)
        check_parity(oracle, g, residual, 2, oracle.schedule(0.01, 2, 0.25), out, label=f"{kind} d={d} ec={residual is not None}")


@pytest.mark.parametrize("d", [ONE_BLOCK, ONE_BLOCK + 1])
@pytest.mark.parametrize("dist", [0, 1, 2])
@pytest.mark.parametrize("kind", ["nan", "inf", "zero", "constant", "denormal", "one"])
def test_special_inputs_on_both_sides_of_the_one_block_limit(oracle, d, dist, kind):
    rng = np.random.default_rng(7)
    g = (rng.standard_t(3.0, size=d) * 1e-3).astype(np.float32)
    if kind == "nan":
        g[d // 2] = np.nan
    elif kind == "inf":
        g[d - 1] = np.inf
    elif kind == "zero":
        g[:] = 0.0
    elif kind == "constant":
        g = np.where(rng.uniform(size=d) < 0.5, -1e-3, 1e-3).astype(np.float32)
    elif kind == "denormal":
        g = (g * 1e-37).astype(np.float32)
    else:
        g[:] = 0.0
        g[d // 3] = 1.0
    for ratios in ([0.01], oracle.schedule(0.01, 3, 0.25)):
        out = run_gpu(g, np.zeros(d, np.float32), dist, ratios)
        check_parity(oracle, g, np.zeros(d, np.float32), dist, ratios, out, label=f"{kind} d={d} dist={dist} M={len(ratios)}")


def test_which_calls_one_block_takes():
    import paper_2101_10761_amd as sidco
    g = np.random.default_rng(1).standard_normal(ONE_BLOCK + 1).astype(np.float32)
    sidco.sidco_set_profiling(True)
    try:
        run_gpu(g[:ONE_BLOCK], None, 0, [0.25, 0.04])
        assert [n for n, _ in sidco.sidco_get_profile()] == ["k_small"]
        run_gpu(g, None, 0, [0.25, 0.04])
        assert [n for n, _ in sidco.sidco_get_profile()] == ["k_fit", "k_compact_dense", "k_final_lists"]
    finally:
        sidco.sidco_set_profiling(False)


@pytest.mark.parametrize("dist,ratios,cap,offset", [(0, [0.25, 0.4], None, 0), (0, [0.25, 0.64, 0.64], 1_000_001, 3),
                                                    (2, [0.4, 0.25], None, 31), (1, [0.3, 0.3], None, 1)])
def test_last_stage_on_the_dense_vector(oracle, dist, ratios, cap, offset):
    """From 50 M elements and a ratio of 0.08 the last stage reads the dense vector and writes the residual back whole."""
    import paper_2101_10761_amd as sidco
    d = 50_000_003
    rng = np.random.default_rng(dist + len(ratios))
    g = rng.standard_normal(d, dtype=np.float32) * np.float32(1e-3)
    r = rng.standard_normal(d, dtype=np.float32) * np.float32(3e-4)
    sidco.sidco_set_profiling(True)
    try:
        out = run_gpu(g, r, dist, ratios, cap=cap, grad_offset=offset, res_offset=offset)
        assert [n for n, _ in sidco.sidco_get_profile()][-1] == "k_select_dense"
    finally:
        sidco.sidco_set_profiling(False)
    check_parity(oracle, g, r, dist, ratios, out, capacity=cap, label=f"dist={dist} {ratios} cap={cap}")


@pytest.mark.parametrize("kind", ["nan", "zero"])
def test_last_stage_on_a_dense_vector_of_nothing_to_select(oracle, kind):
    d = 50_000_000
    g = np.zeros(d, np.float32)
    if kind == "nan":
        g[d // 2] = np.nan
        g[-1] = 3.0
    out = run_gpu(g, np.zeros(d, np.float32), 0, [0.25, 0.4], cap=1000)
    check_parity(oracle, g, np.zeros(d, np.float32), 0, [0.25, 0.4], out, capacity=1000, label=kind)


@pytest.mark.parametrize("sizes,sums", [([1_100_001] * 11 + [1, 300], 564), ([4_160_000] * 3, 2040), ([4_180_000] * 3, 2052),
                                        ([4_180_000, 4_220_000, 4_180_000, 5], 2064)],
                         ids=["short", "below_the_limit", "just_above", "above_the_limit"])
@pytest.mark.parametrize("dist,delta,stages", [(0, 0.02, 1), (1, 0.002, 2), (2, 0.01, 3)])
def test_flat_batches_with_and_without_a_fold_kernel(oracle, sizes, sums, dist, delta, stages):
    """2048 partial sums of a tensor are the most that the first stage's prologue adds up by itself."""
    from test_gpu_batched import check_batched, run_batched
    assert batch_plan(sizes)[1] == sums
    rng = np.random.default_rng(len(sizes) + dist)
    offs = [0] + [int(v) for v in np.cumsum(sizes)]
    g = (rng.standard_t(3.0, size=offs[-1]) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=offs[-1]).astype(np.float32)
    out = run_batched(g, r, offs, delta, dist, stages, repeat=2)
    check_batched(oracle, g, r, offs, delta, dist, stages, out, f"{len(sizes)} tensors dist={dist} M={stages}")


@pytest.mark.parametrize("d,offset", [(ONE_BLOCK + 1, 31), (145 * 256 - 16, 16), (ROUND + 257, 0), (2 * ROUND - 255, 5)])
@pytest.mark.parametrize("dist,ratios", [(0, [0.1]), (2, [0.25, 0.3]), (1, [0.25, 0.45, 0.45]), (0, [0.5, 0.9])])
def test_calls_that_clear_much_of_the_residual(oracle, d, offset, dist, ratios):
    """Their last pass over the vector reads with ordinary loads; lists from the first, the second and the last stage."""
    rng = np.random.default_rng(d + len(ratios))
    g = rng.laplace(0, 1e-3, size=d).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=d).astype(np.float32)
    out = run_gpu(g, r, dist, ratios, grad_offset=offset, res_offset=offset)
    check_parity(oracle, g, r, dist, ratios, out, label=f"d={d} dist={dist} {ratios}")


@pytest.mark.parametrize("d", [20_000_000 - 1, 20_000_000, 20_000_003])
@pytest.mark.parametrize("offset", [(0, 0), (3, 1)])
def test_flat_first_pass_of_calls_that_clear_much_of_the_residual(oracle, d, offset):
    """Such calls take the first pass in address order from 20 M elements, not from 58 M."""
    rng = np.random.default_rng(d)
    g = rng.standard_normal(d, dtype=np.float32) * np.float32(1e-3)
    r = rng.standard_normal(d, dtype=np.float32) * np.float32(3e-4)
    for dist, ratios in ((0, [0.1]), (1, [0.25, 0.3])):
        out = run_gpu(g, r, dist, ratios, grad_offset=offset[0], res_offset=offset[1])
        check_parity(oracle, g, r, dist, ratios, out, label=f"d={d} dist={dist} {ratios} offsets {offset}")


@pytest.mark.parametrize("d,ratios,last", [(50_000_003, [0.25, 0.32], "k_final_lists"), (50_000_003, [0.25, 0.62, 0.62], "k_final_lists"),
                                           (59_999_999, [0.25, 0.35], "k_final_lists"), (60_000_000, [0.25, 0.33], "k_select_dense"),
                                           (62_000_001, [0.25, 0.4], "k_select_dense")])
def test_which_last_stages_read_the_dense_vector(oracle, d, ratios, last):
    """Below 60 M elements lists serve up to a ratio of 0.09 with two stages and 0.1 with more, beyond it up to 0.08."""
    import paper_2101_10761_amd as sidco
    rng = np.random.default_rng(len(ratios))
    g = rng.standard_normal(d, dtype=np.float32) * np.float32(1e-3)
    r = rng.standard_normal(d, dtype=np.float32) * np.float32(3e-4)
    sidco.sidco_set_profiling(True)
    try:
        out = run_gpu(g, r, 0, ratios)
        assert [n for n, _ in sidco.sidco_get_profile()][-1] == last
    finally:
        sidco.sidco_set_profiling(False)
    check_parity(oracle, g, r, 0, ratios, out, label=f"d={d} {ratios}")


def test_a_dense_last_stage_leaves_no_threshold_hint(oracle):
    """The call after it has the same shape and, without a residual, writes candidate lists: with what the workspace held
    before for a hint (10: the lists would start close to the stage's own target) a Gaussian vector falls back."""
    import torch
    import paper_2101_10761_amd as sidco
    d, ratios = 50_000_003, [0.25, 0.4]
    g = np.random.default_rng(1).standard_normal(d, dtype=np.float32)
    ws = torch.full((sidco.sidco_workspace_bytes(d) // 4,), 10.0, dtype=torch.float32, device="cuda:0").view(torch.uint8)
    sidco.sidco_set_workspace(ws)
    try:
        run_gpu(g, np.zeros(d, np.float32), 0, ratios)
        out = run_gpu(g, None, 0, ratios)
    finally:
        sidco.sidco_set_workspace(None)
    assert not out.status & sidco.ST_FALLBACK
    check_parity(oracle, g, None, 0, ratios, out, label="after a dense last stage")


@pytest.mark.parametrize("d", [145 * 256 + k for k in (-31, -16, -1, 0, 1, 225)])
@pytest.mark.parametrize("grad_offset,res_offset", [(5, 5), (16, 16), (31, 31), (0, 30), (29, 4)])
def test_few_tiles_off_the_line_grid(oracle, d, grad_offset, res_offset):
    """Vectors just too long for one block: as many waves as tiles, which end before, on and after the last element."""
    assert d > ONE_BLOCK
    rng = np.random.default_rng(d + 100 * grad_offset + res_offset)
    g = (rng.standard_t(3.0, size=d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=d).astype(np.float32)
    for residual, dist, stages in ((r, 2, 3), (r, 1, 1), (None, 0, 2)):
        ratios = oracle.schedule(0.01, stages, 0.25)
        out = run_gpu(g, residual, dist, ratios, grad_offset=grad_offset, res_offset=res_offset)
        check_parity(oracle, g, residual, dist, ratios, out, label=f"d={d} offsets {grad_offset},{res_offset} M={stages}")


@pytest.mark.parametrize("d", [1, 5, 31, 225, 226, 255, 256, 257, 287, 481, 511, 8 * 256 + 1])
@pytest.mark.parametrize("base", [0, 1, 5, 16, 31])
def test_one_and_two_tiles_in_a_batch_of_one_tensor(oracle, d, base):
    """A batch keeps to tiles however short its tensors are."""
    from test_gpu_batched import check_batched, run_batched
    rng = np.random.default_rng(d + 100 * base)
    g = (rng.standard_t(3.0, size=d) * 1e-3).astype(np.float32)
    r = rng.laplace(0, 3e-4, size=d).astype(np.float32)
    for residual, dist, stages in ((r, 2, 3), (None, 0, 1)):
        out = run_batched(g, residual, [0, d], 0.05, dist, stages, base_offset=base)
        check_batched(oracle, g, residual, [0, d], 0.05, dist, stages, out, f"d={d} base {base} M={stages}")


@pytest.mark.parametrize("dist,stages,offset", [(0, 2, (1, 3)), (1, 2, (0, 31)), (2, 3, (5, 16))])
def test_flat_first_pass_of_single_vectors(oracle, dist, stages, offset):
    """From 58 M elements the first pass runs in address order: every law, gradient and residual off the line grid."""
    d = 58_000_003
    rng = np.random.default_rng(dist)
    g = rng.standard_normal(d, dtype=np.float32) * np.float32(1e-3)
    r = rng.standard_normal(d, dtype=np.float32) * np.float32(3e-4)
    ratios = oracle.schedule(0.001, stages, 0.25)
    out = run_gpu(g, r, dist, ratios, grad_offset=offset[0], res_offset=offset[1])
    check_parity(oracle, g, r, dist, ratios, out, label=f"flat dist={dist} offsets {offset}")


@pytest.mark.parametrize("dist", [0, 1, 2])
@pytest.mark.parametrize("value,at", [(np.nan, 0), (np.inf, -1), (-np.inf, 29_000_000)])
def test_non_finite_values_in_a_flat_first_pass(oracle, dist, value, at):
    """One of them makes the first stage's sums non-finite: nothing is selected, the residual takes the sum."""
    d = 58_000_001
    g = np.full(d, 1e-3, np.float32)
    g[at] = value
    r = np.zeros(d, np.float32)
    out = run_gpu(g, r, dist, [0.25, 0.04], res_offset=1)
    assert out.count == 0 and np.isnan(out.eta) and out.status & 1
    check_parity(oracle, g, r, dist, [0.25, 0.04], out, label=f"{value} at {at} dist={dist}")


@pytest.mark.parametrize("d", [44_999_999, 45_000_001])
@pytest.mark.parametrize("dist,offset", [(0, 0), (2, 7)])
def test_sums_only_stages_without_a_residual(oracle, d, dist, offset):
    """Calls of three stages whose first only sums read with ordinary loads from 45 M elements."""
    rng = np.random.default_rng(d + dist)
    g = rng.standard_normal(d, dtype=np.float32) * np.float32(1e-3)
    ratios = oracle.schedule(0.06, 3, 0.25)
    out = run_gpu(g, None, dist, ratios, grad_offset=offset)
    check_parity(oracle, g, None, dist, ratios, out, label=f"d={d} dist={dist} offset {offset}")
