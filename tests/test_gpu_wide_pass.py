"""GPU parity of calibrations of more than 16 columns on bf16 models, which run as one wide pass: against the oracle,
sequence by sequence, and against the same calibration run in passes of at most 16 columns (EASYSPEC_PAIR_PASSES=0;
same precision, other summation order: the oracle tolerance).  Column counts at the edges of the column tiles (17, 32,
33), of the column blocks (128, 129) and of the range (256); ragged token counts, idle sequences, fuzzy slots to drop,
contexts of one and of several chunks; next tokens, logits of last rows and of all rows, caches, lengths, hidden rows.
Every kernel that a cut of a product can choose is run, and each case asserts the cuts it is there for: (row tiles per
wave, column tiles, column blocks)."""
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


def run_case(oracle, gpu, monkeypatch, cfg, seed, ctxs, n_calib, max_calib, all_rows, check=None, fuzzy_first=1, cuts=None):
    """check: the sequences compared with the oracle (default: all).  cuts: what the products' cuts have to be."""
    import torch
    import paper_2502_02493_amd as es
    B = len(ctxs)
    for op, want in (cuts or {}).items():
        r = es.easyspec_wide_walk(es.make_config(cfg, B, 64, max_calib), getattr(es, "EASYSPEC_OP_" + op), sum(n_calib))
        assert (r["row_tiles"], r["col_tiles"], r["col_blocks"]) == want, (op, r)
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


@pytest.mark.parametrize("shape,n_calib,ctxs,all_rows,cut", [
    ("tiny", [16, 1], [40, 300], True, (2, 2, 1)),                                     # 17: the second column tile holds one column
    ("tiny", [9, 0, 16, 7], [33, 5, 257, 64], False, (2, 2, 1)),                       # 32, one sequence idle
    ("tiny_qwen", [11, 11, 11], [9, 320, 63], True, (2, 3, 1)),                        # 33: three tiles; biases, 7 heads per KV head
    ("tiny_qwen", [16, 5, 16, 16, 3], [100, 2, 258, 31, 64], False, (2, 4, 1)),        # 56
    ("tiny", [16, 15, 14, 13, 12, 11], [20, 70, 257, 3, 129, 64], True, (4, 3, 2)),    # 81: six tiles in two blocks, four row tiles per wave
])
def test_small_models(oracle, gpu, monkeypatch, shape, n_calib, ctxs, all_rows, cut):
    run_case(oracle, gpu, monkeypatch, synth.model_shape(shape, dtype="bf16"), 1300 + sum(n_calib), ctxs, n_calib, 16, all_rows,
             cuts={op: cut for op in ("QKV", "OPROJ", "GATEUP", "DOWN", "HEAD")})


@pytest.mark.parametrize("total,split,whole", [(112, (4, 4, 2), (4, 3, 3)), (128, (4, 4, 2), (4, 3, 3)), (129, (4, 5, 2), (4, 3, 3)),
                                               (177, (4, 6, 2), (4, 3, 4)), (200, (4, 8, 2), (4, 4, 4)), (256, (4, 8, 2), (4, 4, 4))])
def test_column_blocks(oracle, gpu, monkeypatch, total, split, whole):
    """Products whose K may be split: two blocks of four, five (129 fills one column of the ninth tile), six and eight column
    tiles; gate/up and the head of a small model: three and four blocks of three and four."""
    n = [16] * (total // 16) + ([total % 16] if total % 16 else [])
    ctxs = [(37 * i) % 290 + 1 for i in range(len(n))]
    run_case(oracle, gpu, monkeypatch, synth.model_shape("tiny", dtype="bf16"), 1400 + total, ctxs, n, 16, total == 129,
             check=[0, len(n) // 2, len(n) - 1], cuts=dict(QKV=split, OPROJ=split, DOWN=split, GATEUP=whole, HEAD=whole))


@pytest.mark.parametrize("n_seq,cut", [(5, (4, 5, 1)), (6, (4, 6, 1)), (8, (4, 8, 1))])
def test_head_of_all_rows_in_one_block(oracle, gpu, monkeypatch, n_seq, cut):
    """A vocabulary whose row blocks fill the CUs: the logits of every column from one block of five, six and eight tiles."""
    ctxs = [(53 * i) % 280 + 1 for i in range(n_seq)]
    run_case(oracle, gpu, monkeypatch, synth.model_shape("tiny", dtype="bf16", vocab=65536), 1700 + n_seq, ctxs, [16] * n_seq, 16, True,
             check=[0, n_seq - 1], cuts=dict(HEAD=cut))


@pytest.mark.parametrize("n_calib,layers,cut", [([6, 6, 6, 6], 3, (2, 2, 1)), ([16, 16, 3, 16, 16], 3, (4, 3, 2)), ([16] * 16, 5, (4, 8, 2))])
def test_8b_layer_shape(oracle, gpu, monkeypatch, n_calib, layers, cut):
    """The 8B layer shape (packed tiles of 14 and 12 rows, split K): 24, 67 and 256 columns."""
    cfg = synth.model_shape("llama3_8b", n_layers=layers, vocab=4096)
    ctxs = ([300, 40, 700, 129, 8] + [90 + 41 * i for i in range(11)])[:len(n_calib)]
    run_case(oracle, gpu, monkeypatch, cfg, 1500 + sum(n_calib), ctxs, n_calib, 16, False, check=[0, 2], cuts=dict(GATEUP=cut))


@pytest.mark.parametrize("n_seq,cut", [(5, (4, 5, 1)), (6, (4, 6, 1)), (16, (4, 6, 3))])
def test_qwen2_7b_layer_shape(oracle, gpu, monkeypatch, n_seq, cut):
    """The Qwen2-7B layer shape (biases, 7 heads of 128 elements per KV head, 18 944 rows of gate and up) at 3 layers:
    80, 96 and 256 columns."""
    cfg = synth.model_shape("qwen2_7b", n_layers=3, vocab=4096)
    ctxs = [(211 * i) % 700 + 20 for i in range(n_seq)]
    run_case(oracle, gpu, monkeypatch, cfg, 1750 + n_seq, ctxs, [16] * n_seq, 16, False, check=[0, 3], cuts=dict(GATEUP=cut))


def test_head_dim_128_one_head_per_kv(oracle, gpu, monkeypatch):
    cfg = synth.model_shape("tiny", dtype="bf16", head_dim=128, n_q_heads=2, n_kv_heads=2, vocab=1003)
    run_case(oracle, gpu, monkeypatch, cfg, 1600, [67, 1, 400], [7, 16, 10], 16, True)
