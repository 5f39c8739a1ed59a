"""GPU parity of fuzzy steps of batches whose contexts differ (the vector attention kernel's grid then lists every column's
own chunks instead of the longest column's for all): 1, 2, 4 and 7 query heads per KV head, heads of 64 and 128 elements,
contexts from one slot to several chunks, sixteen sequences, forced chunk counts."""
import numpy as np
import pytest

import easyspec_synth as synth
from tolerances import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,ctxs,nch", [
    (dict(name="tiny", dtype="fp32"), [300, 1, 77, 513], 0),
    (dict(name="tiny", dtype="bf16"), [5, 700, 260, 31, 64], 7),
    (dict(name="tiny_qwen", dtype="bf16"), [600, 40, 333], 0),
    (dict(name="tiny", dtype="bf16", head_dim=128, n_q_heads=8, n_kv_heads=2), [1000, 17, 400, 256], 13),
    (dict(name="tiny", dtype="bf16", head_dim=128, n_q_heads=2, n_kv_heads=2), [50 * i + 1 for i in range(16)], 0),
])
def test_draft_step(oracle, monkeypatch, model, ctxs, nch):
    import torch
    assert torch.cuda.is_available()
    import gpu_harness as gpu
    if nch:
        monkeypatch.setenv("EASYSPEC_ATTN_NCH", str(nch))
    cfg = synth.model_shape(**model)
    B, bounds = len(ctxs), np.array([0, 1, 3, cfg["n_layers"]], np.int32)
    w = synth.make_weights(cfg, 1700)
    om = oracle.Model(cfg, w, max(ctxs) + 8)
    toks = synth.make_tokens(1701, 2 * B, cfg["vocab"]).reshape(2, B)
    g = gpu.GpuDrafter(cfg, w, max_batch=B, max_ctx=max(ctxs) + 8, max_calib=1)
    try:
        g.set_groups(bounds)
        seqs = []
        for b, n in enumerate(ctxs):
            k, v = synth.make_kv_prefix(cfg, 1702, n, seq=b)
            g.import_kv(b, k, v)
            seqs.append(oracle.Sequence(om))
            seqs[-1].import_kv(k, v)
        for step in range(2):
            _, logits = g.draft_step({b: int(toks[step, b]) for b in range(B)})
            for b in range(B):
                gpu.assert_close(logits[b], seqs[b].fuzzy_step(bounds, int(toks[step, b])), TOL[cfg["dtype"]], f"sequence {b}, step {step}")
    finally:
        g.close()
