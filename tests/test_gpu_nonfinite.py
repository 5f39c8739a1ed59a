"""A token whose activations are not finite (its embedding row holds a NaN) spoils what sees it and nothing else: the tokens
before it, other sequences and their cache entries keep the values they have without it, on every route that a calibration
takes (the matrix-core kernel multiplies slots that a row does not see by probabilities of zero)."""
import numpy as np
import pytest

import easyspec_synth as synth
from tolerances import TOL

pytestmark = pytest.mark.gpu
BAD = 7  # the token id whose embedding row is spoilt


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device; none is visible")
    import gpu_harness
    return gpu_harness


ROUTES = {"wide": {}, "passes of 16, vector kernel": dict(EASYSPEC_PAIR_PASSES="0", EASYSPEC_ATTN_MFMA="0"),
          "passes of 16, matrix cores": dict(EASYSPEC_PAIR_PASSES="0", EASYSPEC_ATTN_MFMA="2")}


def run(gpu, cfg, w, ctxs, toks):
    g = gpu.GpuDrafter(cfg, w, max_batch=len(ctxs), max_ctx=max(ctxs) + 64, max_calib=16)
    try:
        for b, n in enumerate(ctxs):
            k, v = synth.make_kv_prefix(cfg, 1801, n, seq=b)
            g.import_kv(b, k, v)
        _, lg = g.calibrate(toks)
        return lg, {b: g.export_kv(b, ctxs[b] + len(toks[b])) for b in toks}
    finally:
        g.close()


def both(gpu, cfg, ctxs, toks):
    w = synth.make_weights(cfg, 1800)
    clean = run(gpu, cfg, w, ctxs, toks)
    w["embed"] = w["embed"].copy()
    w["embed"][BAD, 3] = 0x7FC0  # a bf16 NaN
    return clean, run(gpu, cfg, w, ctxs, toks)


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("shape,ctxs", [("tiny", [40, 333, 61]), ("tiny_qwen", [5, 270, 129]), ("hd128", [700, 64, 20])])
def test_calibration(gpu, monkeypatch, route, shape, ctxs):
    for k, v in ROUTES[route].items():
        monkeypatch.setenv(k, v)
    cfg = synth.model_shape("tiny", dtype="bf16", head_dim=128, n_q_heads=8, n_kv_heads=2) if shape == "hd128" else synth.model_shape(shape, dtype="bf16")
    t = synth.make_tokens(1802, 64, cfg["vocab"])
    toks = {0: [int(x) for x in t[:9]], 1: [int(x) for x in t[16:32]], 2: [int(x) for x in t[40:43]]}
    toks = {b: [x if x != BAD else BAD + 1 for x in v] for b, v in toks.items()}
    toks[0][5] = toks[1][15] = BAD  # in the middle of one sequence, at the end of another; the third has none
    (lg0, kv0), (lg1, kv1) = both(gpu, cfg, ctxs, toks)
    for b, ok in ((0, 5), (1, 15), (2, 3)):
        gpu.assert_close(lg1[b][:ok], lg0[b][:ok], TOL["bf16"], f"{route}: sequence {b}, tokens before the spoilt one")
        assert np.isnan(lg1[b][ok:]).all()
        for x1, x0 in zip(kv1[b], kv0[b]):
            gpu.assert_close(x1[:, :, :ctxs[b] + ok], x0[:, :, :ctxs[b] + ok], TOL["bf16"], f"{route}: cache of sequence {b}")
