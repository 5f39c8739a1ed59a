"""What a one-launch pass of a small model that gave up waiting does to its context (include/easyspec.h, Conventions): every entry
point that uses or hands out the context's state refuses, whatever route the call would take, and another context is untouched.
The give-up is forced from the host, which picks the kernel whose own bounded wait has a limit of one poll; it ends normally."""
import numpy as np
import pytest

import easyspec_synth as synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device; none is visible")
    import gpu_harness
    return gpu_harness


@pytest.fixture
def pair(gpu):
    """Two contexts of the same model after the same prompt, and a stream."""
    import torch
    cfg = synth.model_shape("tiny")
    w = synth.make_weights(cfg, 2200)
    st = torch.cuda.Stream()
    gs = []
    try:
        with torch.cuda.stream(st):
            for _ in range(2):
                gs.append(gpu.GpuDrafter(cfg, w, max_batch=2, max_ctx=400, max_calib=16, stream=st.cuda_stream))
                gs[-1].calibrate({0: [1, 2, 3, 4]})
        yield gs[0], gs[1], st
    finally:
        for g in gs:
            g.close()


def refuses(fn, *a):
    import paper_2502_02493_amd as es
    with pytest.raises(es.EasySpecError) as e:
        fn(*a)
    assert e.value.code == es.EASYSPEC_EHIP and "gave up" in str(e.value), e.value


def refuses_everything(g, monkeypatch):
    import torch
    import paper_2502_02493_amd as es
    cfg, c = g.cfg, g.ctx
    k = np.zeros((cfg["n_layers"], cfg["n_kv_heads"], 4, cfg["head_dim"]), np.float32)
    hid = torch.zeros(16, cfg["d_model"], device="cuda")
    for env in (None, "0"):                                       # the route of the failed pass and the launches
        if env:
            monkeypatch.setenv("EASYSPEC_RESIDENT", env)
        refuses(es.easyspec_draft_step, c, g.tok_in, g.tok_out, g.logits)
        refuses(g.draft_tree_step, {0: ([1], [-1])})
        refuses(es.easyspec_calibrate, c, g.calib_tok, [1, 0], g.tok_out, g.logits, 0)
    monkeypatch.delenv("EASYSPEC_RESIDENT")
    g.set_full_layer(True)
    refuses(es.easyspec_draft_step, c, g.tok_in, g.tok_out, g.logits)
    refuses(es.easyspec_get_lens, c, 2)
    refuses(es.easyspec_truncate, c, 0, 0)
    refuses(es.easyspec_kv_import, c, 1, k, k, 4)
    refuses(es.easyspec_kv_export, c, 0, k, k, 4)
    refuses(es.easyspec_get_hidden, c, hid, 16)


def test_every_entry_point_refuses(pair, monkeypatch):
    import paper_2502_02493_amd as es
    a, b, st = pair
    want = b.draft_step({0: 9})[1]
    es.easyspec_force_give_up(a.ctx, 1)
    es.easyspec_draft_step(a.ctx, a.tok_in, a.tok_out, a.logits)  # gives up; returns before it does
    st.synchronize()
    refuses_everything(a, monkeypatch)
    es.easyspec_force_give_up(a.ctx, 0)                           # for good: what the pass left behind stays wrong
    refuses(es.easyspec_get_lens, a.ctx, 2)
    es.easyspec_truncate(b.ctx, 0, 4)
    assert np.array_equal(b.draft_step({0: 9})[1], want)           # the other context goes on


@pytest.mark.parametrize("entry", ["export", "import", "profile_end"])
def test_calls_that_synchronise_look_again(pair, entry):
    """No synchronisation between the pass and the call: it may find out only after its own."""
    import paper_2502_02493_amd as es
    a, _, _ = pair
    k = np.zeros((a.cfg["n_layers"], a.cfg["n_kv_heads"], 4, a.cfg["head_dim"]), np.float32)
    es.easyspec_force_give_up(a.ctx, 1)
    es.easyspec_draft_step(a.ctx, a.tok_in, a.tok_out, a.logits)
    if entry == "profile_end":
        es.easyspec_profile_begin(a.ctx, es.EASYSPEC_OP_ALL, 4)
        refuses(es.easyspec_profile_end, a.ctx)
    elif entry == "export":
        refuses(es.easyspec_kv_export, a.ctx, 0, k, k, 4)
    else:
        refuses(es.easyspec_kv_import, a.ctx, 1, k, k, 4)


def test_a_replayed_pass(pair, monkeypatch):
    import torch
    import paper_2502_02493_amd as es
    a, _, st = pair
    graph = torch.cuda.CUDAGraph()
    es.easyspec_force_give_up(a.ctx, 1)
    with torch.cuda.graph(graph, stream=st):
        es.easyspec_draft_step(a.ctx, a.tok_in, a.tok_out, a.logits)
    es.easyspec_force_give_up(a.ctx, 0)
    with torch.cuda.stream(st):
        a.draft_step({0: 5})                                       # a pass with the ordinary limit: all is well
        graph.replay()
    st.synchronize()
    refuses_everything(a, monkeypatch)


@pytest.mark.parametrize("over", [dict(head_dim=128, n_kv_heads=2), dict(dtype="bf16"), dict(n_kv_heads=1)])
def test_models_without_such_a_kernel(gpu, over):
    import paper_2502_02493_amd as es
    cfg = synth.model_shape("tiny", **over)
    g = gpu.GpuDrafter(cfg, synth.make_weights(cfg, 2201), max_batch=1, max_ctx=64, max_calib=16)
    try:
        with pytest.raises(es.EasySpecError) as e:
            es.easyspec_force_give_up(g.ctx, 1)
        assert e.value.code == es.EASYSPEC_EINVAL
        assert np.isfinite(g.calibrate({0: [1, 2, 3]})[1][0]).all()
        assert int(g.lens()[0][0]) == 3
    finally:
        g.close()
