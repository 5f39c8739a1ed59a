"""GPU parity of the matrix-core attention kernel with one, two and four tiles of 16 query rows per workgroup (the
library takes as many as the longest run of columns of one sequence fills): calibrations of 16 and 5 + 9 tokens and
tree levels, contexts around the 64-slot super tile and over several chunks, 1, 2, 4 and 7 query heads per KV head
(7: tiles whose rows are no multiple of the heads; a wave without rows where 3 of 4 tiles are filled)."""
import pytest

import easyspec_synth as synth
from test_gpu_parity import iteration_parity
from test_gpu_tree import tree_parity
from test_gpu_attn_mfma import test_calibration_of_two_sequences_in_one_call as _two_sequences

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device; none is visible")
    import gpu_harness
    return gpu_harness


@pytest.fixture(params=[1, 2, 4])
def tiles(request, monkeypatch):
    monkeypatch.setenv("EASYSPEC_ATTN_MFMA", "2")
    monkeypatch.setenv("EASYSPEC_ATTN_ROW_TILES", str(request.param))
    return request.param


@pytest.mark.parametrize("model,bounds,prompt", [
    (dict(name="tiny"), [0, 1, 3, 4], 64),
    (dict(name="tiny"), [0, 4], 321),
    (dict(name="tiny_qwen"), [0, 1, 4, 5], 290),
    (dict(name="tiny", head_dim=128, n_q_heads=4, n_kv_heads=1), [0, 1, 3, 4], 129),
    (dict(name="tiny", head_dim=128, n_q_heads=2, n_kv_heads=2), [0, 1, 3, 4], 65),
])
def test_iteration(oracle, gpu, tiles, model, bounds, prompt):
    iteration_parity(oracle, gpu, synth.model_shape(dtype="bf16", **model), 1200 + prompt, bounds, prompt, 4, n_iters=1)


@pytest.mark.parametrize("shape,widths", [("tiny", [3, 5, 12]), ("tiny_qwen", [2, 9])])
def test_tree(oracle, gpu, tiles, shape, widths):
    cfg = synth.model_shape(shape, dtype="bf16")
    tree_parity(oracle, gpu, cfg, 1210, [0, 1, cfg["n_layers"]], 270, widths)


def test_two_sequences(oracle, gpu, tiles):
    _two_sequences(oracle, gpu)
