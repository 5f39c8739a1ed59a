"""The end of a weight kernel's tile (a thread per element behind the waves' partial sums) where a workgroup has fewer threads than
the tile has elements: one and two waves with up to 16 columns (256 elements), tiles of 12 and 14 rows, one and two row tiles per
workgroup, chain steps, calibrations and tree levels, against the oracle."""
import pytest

import easyspec_synth as synth
from test_gpu_parity import iteration_parity
from test_gpu_tree import tree_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device; none is visible")
    import gpu_harness
    return gpu_harness


@pytest.fixture(params=[1, 2, 8])
def waves(request, monkeypatch):
    for op in ("QKV", "O", "GU", "DOWN", "HEAD"):
        monkeypatch.setenv(f"EASYSPEC_NW_{op}", str(request.param))
    return request.param


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("pair", [None, "1"])
def test_iteration(oracle, gpu, monkeypatch, waves, dtype, pair):
    if pair and dtype == "bf16":
        monkeypatch.setenv("EASYSPEC_PAIR_TILES", pair)
        monkeypatch.setenv("EASYSPEC_TILE_ROWS", "14")
        monkeypatch.setenv("EASYSPEC_QKV_TILE_ROWS", "12")
    cfg = synth.model_shape("tiny_qwen", dtype=dtype)
    iteration_parity(oracle, gpu, cfg, 1300, [0, 1, 4, 5], 33, 4, n_iters=1)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_tree(oracle, gpu, waves, dtype):
    cfg = synth.model_shape("tiny", dtype=dtype)
    tree_parity(oracle, gpu, cfg, 1310, [0, 1, 3, 4], 40, [1, 9, 16])


def test_most_partial_sums(gpu, monkeypatch):
    """Sixteen waves of four row tiles: 80 KB of partial sums, more than a launch has unasked.  Against eight waves, on one layer, whose
    cache entries do not depend on them: gate/up sums of 4096 products in another order (2^-24 sqrt(4096) of a sum at most), activations
    in two bf16 terms that may round the other way (2^-17 of one), both averaged by the sums that follow."""
    import paper_2502_02493_amd as es
    cfg = synth.model_shape("tiny", dtype="bf16", n_layers=1, d_model=4096, vocab=256)
    w = synth.make_weights(cfg, 1320)
    toks = {0: [int(t) for t in synth.make_tokens(1321, 16, cfg["vocab"])]}
    monkeypatch.setenv("EASYSPEC_PAIR_TILES", "1")
    got = []
    for waves in (16, 8):
        monkeypatch.setenv("EASYSPEC_NW_GU", str(waves))
        plan = es.easyspec_weight_walk(es.make_config(cfg, 1, 64, 16), es.EASYSPEC_OP_GATEUP, 16, 1)
        assert (plan["waves"], plan["units_per_wg"], plan["fragments"]) == (waves, 2, 2)
        g = gpu.GpuDrafter(cfg, w, max_batch=1, max_ctx=64, max_calib=16)
        try:
            got.append(g.calibrate(toks, all_rows=True)[1][0])
        finally:
            g.close()
    gpu.assert_close(got[0], got[1], 1e-5, "sixteen and eight waves")
