"""GPU parity of calibrations of more than 16 columns on bf16 models, which run as one wide pass: against the oracle,
sequence by sequence, and against the same calibration run in passes of at most 16 columns (EASYSPEC_PAIR_PASSES=0;
same precision, other summation order: the oracle tolerance).  Column counts at the edges of the column tiles (17, 32,
33), of the column blocks (128, 129) and of the range (256); ragged token counts, idle sequences, fuzzy slots to drop,
contexts of one and of several chunks; next tokens, logits of last rows and of all rows, caches, lengths, hidden rows."""
import numpy as np
import pytest

import easyspec_synth as synth
from tolerances import TOL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device; none is visible")
    import gpu_harness
    return gpu_harness


def run_case(oracle, gpu, monkeypatch, cfg, seed, ctxs, n_calib, max_calib, all_rows, check=None, fuzzy_first=1):
    """check: the sequences compared with the oracle (default: all)."""
    import torch
    import paper_2502_02493_amd as es
    B = len(ctxs)
    w = synth.make_weights(cfg, seed)
    max_ctx = max(ctxs) + fuzzy_first + max_calib + 8
    toks = synth.make_tokens(seed + 1, B * (max_calib + fuzzy_first), cfg["vocab"]).reshape(B, -1)
    calib = {b: [int(t) for t in toks[b, fuzzy_first:fuzzy_first + n]] for b, n in enumerate(n_calib) if n > 0}
    assert sum(n_calib) > 16
    bounds = np.array([0, 1, cfg["n_layers"] - 1, cfg["n_layers"]], np.int32)
    results = []
    for env in (None, "0"):
        if env is None:
            monkeypatch.delenv("EASYSPEC_PAIR_PASSES", raising=False)
        else:
            monkeypatch.setenv("EASYSPEC_PAIR_PASSES", env)
        g = gpu.GpuDrafter(cfg, w, max_batch=B, max_ctx=max_ctx, max_calib=max_calib)
        try:
            g.set_groups(bounds)
            for b, n in enumerate(ctxs):
                k, v = synth.make_kv_prefix(cfg, seed + 2, n, seq=b)
                g.import_kv(b, k, v)
            for step in range(fuzzy_first):
                g.draft_step({b: int(toks[b, step]) for b in range(B)})
            if env is None:
                es.easyspec_poison_workspaces(g.ctx)  # nothing of an earlier pass may be read
            gt, gl = g.calibrate(calib, all_rows=all_rows)
            hid = torch.zeros(16, cfg["d_model"], device="cuda")
            rows = es.easyspec_get_hidden(g.ctx, hid, 16)
            torch.cuda.synchronize()
            kv = {b: g.export_kv(b, ctxs[b] + n_calib[b]) for b in calib}
            # a fuzzy step on the calibrated state
            ft, fl = g.draft_step({b: int(toks[b, 0]) for b in range(B)})
            results.append((gt, gl, kv, g.lens(), hid[:rows].cpu().numpy(), fl))
        finally:
            g.close()
    (gt1, gl1, kv1, lens1, h1, f1), (gt0, gl0, kv0, lens0, h0, f0) = results
    tol = TOL["bf16"]
    kv_tol = max(tol, 2e-3)   # a bf16 entry may differ by one unit in the last place
    assert h1.shape == h0.shape
    gpu.assert_close(h1, h0, tol, "hidden rows")
    for b in gl1:
        gpu.assert_close(gl1[b], gl0[b], tol, f"sequence {b}: wide against passes of 16")
        gpu.assert_close(f1[b], f0[b], tol, f"sequence {b}: fuzzy step after it")
        for x1, x0 in zip(kv1[b], kv0[b]):
            assert gpu.rel_l2(x1, x0) < kv_tol
        last = np.asarray(gl1[b]).reshape(-1, cfg["vocab"])[-1]
        assert gt1[b] == int(np.argmax(last))
    assert np.array_equal(lens1[0], lens0[0]) and np.array_equal(lens1[1], lens0[1])
    model = oracle.Model(cfg, w, max_ctx)
    for b in (range(B) if check is None else check):
        if n_calib[b] == 0:
            continue
        so = oracle.Sequence(model)
        k, v = synth.make_kv_prefix(cfg, seed + 2, ctxs[b], seq=b)
        so.import_kv(k, v)
        for step in range(fuzzy_first):
            so.fuzzy_step(bounds, int(toks[b, step]))
        wl = so.calibrate(calib[b], all_rows=all_rows)
        gpu.assert_close(gl1[b], wl, tol, f"calibration logits, sequence {b}")
        kk, vv = kv1[b]
        assert gpu.rel_l2(kk, so.K[:, :, :so.precise]) < kv_tol
        assert gpu.rel_l2(vv, so.V[:, :, :so.precise]) < kv_tol


@pytest.mark.parametrize("shape,n_calib,ctxs,all_rows", [
    ("tiny", [16, 1], [40, 300], True),                                     # 17: the second column tile holds one column
    ("tiny", [9, 0, 16, 7], [33, 5, 257, 64], False),                       # 32, one sequence idle
    ("tiny_qwen", [11, 11, 11], [9, 320, 63], True),                        # 33: three tiles; biases, 7 heads per KV head
    ("tiny_qwen", [16, 5, 16, 16, 3], [100, 2, 258, 31, 64], False),        # 56
    ("tiny", [16, 15, 14, 13, 12, 11], [20, 70, 257, 3, 129, 64], True),    # 81: six tiles, four row tiles per wave
])
def test_small_models(oracle, gpu, monkeypatch, shape, n_calib, ctxs, all_rows):
    run_case(oracle, gpu, monkeypatch, synth.model_shape(shape, dtype="bf16"), 1300 + sum(n_calib), ctxs, n_calib, 16, all_rows)


@pytest.mark.parametrize("total", [112, 128, 129, 200, 256])
def test_column_blocks(oracle, gpu, monkeypatch, total):
    """Seven and eight column tiles in one block, then two blocks of five, seven and eight tiles (129 fills one column of
    its ninth tile)."""
    n = [16] * (total // 16) + ([total % 16] if total % 16 else [])
    ctxs = [(37 * i) % 290 + 1 for i in range(len(n))]
    run_case(oracle, gpu, monkeypatch, synth.model_shape("tiny", dtype="bf16"), 1400 + total, ctxs, n, 16, total == 129,
             check=[0, len(n) // 2, len(n) - 1])


@pytest.mark.parametrize("n_calib", [[6, 6, 6, 6], [16, 16, 3, 16, 16]])
def test_8b_layer_shape(oracle, gpu, monkeypatch, n_calib):
    """The 8B layer shape (packed tiles of 14 and 12 rows, split K) at 3 layers."""
    cfg = synth.model_shape("llama3_8b", n_layers=3, vocab=4096)
    run_case(oracle, gpu, monkeypatch, cfg, 1500 + sum(n_calib), [300, 40, 700, 129, 8][:len(n_calib)], n_calib, 16, False, check=[0, 2])


def test_head_dim_128_one_head_per_kv(oracle, gpu, monkeypatch):
    cfg = synth.model_shape("tiny", dtype="bf16", head_dim=128, n_q_heads=2, n_kv_heads=2, vocab=1003)
    run_case(oracle, gpu, monkeypatch, cfg, 1600, [67, 1, 400], [7, 16, 10], 16, True)
