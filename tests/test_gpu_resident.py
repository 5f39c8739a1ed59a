"""Passes of small models in one launch (csrc/resident.hip) against the same calls as separate launches (EASYSPEC_RESIDENT=0) and
against the oracle, at the edges of its range: one slot and the longest contexts, one column and the most, every number of query
heads per KV head, row tiles that fill a wave's registers and that leave most of them empty, vocabularies that end inside a tile.
Tolerances: those against the oracle (tests/tolerances.py).  The two routes add up in different orders, so that some bit of an
fp32 result tells them apart: asserted where the route is part of the claim."""
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


def both(monkeypatch, fn):
    monkeypatch.setenv("EASYSPEC_RESIDENT", "0")
    apart = fn()
    monkeypatch.delenv("EASYSPEC_RESIDENT")
    return apart, fn()


def compare(gpu, apart, one, tol, what):
    for i, (a, b) in enumerate(zip(apart, one)):
        assert np.isfinite(np.asarray(a, np.float64)).all()
        gpu.assert_close(b, a, tol, f"{what}: output {i}")


# layers, d_model, query heads, KV heads, d_ffn, vocabulary, columns that one launch takes at a first token
SHAPES = {"one head per KV head": (2, 256, 4, 4, 512, 1000, 16), "four": (3, 128, 8, 2, 96, 17, 12), "eight": (2, 512, 8, 1, 1536, 16384, 3),
          "full registers": (2, 768, 12, 6, 1536, 1600, 6), "seven, odd tiles": (4, 448, 7, 1, 1184, 1001, 9), "one tile": (1, 32, 1, 1, 32, 16, 16)}


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_against_launches(gpu, monkeypatch, shape, dtype):
    L, d, hq, hkv, f, v, most = SHAPES[shape]
    cfg = synth.model_shape("tiny_qwen" if hq % 2 else "tiny", n_layers=L, d_model=d, n_q_heads=hq, n_kv_heads=hkv, d_ffn=f, vocab=v, dtype=dtype)
    w = synth.make_weights(cfg, 2100)
    t = [int(x) for x in synth.make_tokens(2101, 64, v)]
    edge = 320 if dtype == "fp32" else 640
    kv = synth.make_kv_prefix(cfg, 2102, edge - 5)

    def run():
        g = gpu.GpuDrafter(cfg, w, max_batch=3, max_ctx=edge + 40, max_calib=16)
        outs = []
        try:
            _, lg = g.calibrate({2: t[40:40 + most]})                        # as many columns as one launch takes, no pass before it
            outs.append(lg[2])
            g.set_groups([0, L] if L < 3 else [0, 1, L])
            _, lg = g.calibrate({0: t[:1]})                                  # a first token: no cached slot
            outs.append(lg[0])
            _, lg = g.calibrate({0: t[1:1 + most]})                          # ... and behind a slot
            outs += [lg[0], g.hidden()]
            outs.append(g.draft_step({0: t[20]})[1][0])
            g.import_kv(1, *kv)
            _, lg = g.draft_tree_step({1: (t[21:23], [-1, -1])})
            outs.append(lg[1])
            _, lg = g.draft_tree_step({1: (t[23:26], [0, 1, 1])})
            outs.append(lg[1])
            _, lg = g.calibrate({0: t[30:31], 1: t[31:33]})                  # two sequences, one with a token tree to drop
            outs += [lg[0], lg[1]]
            for i in range(3):                                               # the second one ends at the rule's last slot
                outs.append(g.draft_step({0: t[33 + i], 1: t[36 + i]})[1][:2])
            n = int(g.lens()[0][1]) + 3
            assert n == edge
            outs += list(g.export_kv(0, int(g.lens()[0][0]) + 3)) + list(g.export_kv(1, n))
            return outs
        finally:
            g.close()

    apart, one = both(monkeypatch, run)
    kv_tol = TOL[dtype] if dtype == "fp32" else max(TOL[dtype], 2e-3)        # a bf16 entry may differ by one unit in the last place
    compare(gpu, apart[:-4], one[:-4], TOL[dtype], shape)
    compare(gpu, apart[-4:], one[-4:], kv_tol, shape + ", cache")
    assert not np.array_equal(apart[0], one[0]) or d == 32                   # (32: one term per wave, no order to tell apart)


@pytest.mark.parametrize("dtype,calls", [
    ("fp32", ((319, 1, True), (320, 1, False), (100, 9, True), (100, 10, False), (311, 9, True), (312, 9, False))),
    ("bf16", ((639, 1, True), (640, 1, False), (100, 9, True), (100, 10, False), (635, 5, True), (636, 5, False), (634, 6, False)))])
def test_the_edges_of_the_rule(gpu, monkeypatch, dtype, calls):
    """The last context and column count of the one route and the first of the other."""
    cfg = synth.model_shape("tiny_qwen", dtype=dtype)
    w = synth.make_weights(cfg, 2110)
    t = [int(x) for x in synth.make_tokens(2111, 16, cfg["vocab"])]

    def run(ctx, n):
        def fn():
            g = gpu.GpuDrafter(cfg, w, max_batch=1, max_ctx=700, max_calib=16)
            try:
                g.import_kv(0, *synth.make_kv_prefix(cfg, 2112, ctx))
                return g.calibrate({0: t[:n]})[1][0]
            finally:
                g.close()
        return both(monkeypatch, fn)

    for ctx, n, one_launch in calls:
        a, b = run(ctx, n)
        assert np.array_equal(a, b) != one_launch, (ctx, n)
        gpu.assert_close(b, a, TOL[dtype], f"context {ctx}, {n} columns")


# calls inside those limits that the launches do faster: many columns of a large vocabulary, units in several rounds
@pytest.mark.parametrize("dtype,shape,group,most", [("fp32", (2, 544, 4, 2, 864, 9921), 7, 10), ("bf16", (5, 1024, 4, 1, 2176, 13430), 7, 5),
                                                     ("fp32", (19, 576, 6, 3, 608, 613), 7, 10)])
def test_the_cost_rule(gpu, monkeypatch, dtype, shape, group, most):
    import paper_2502_02493_amd as es
    L, d, hq, hkv, f, v = shape
    cfg = synth.model_shape("tiny", n_layers=L, d_model=d, n_q_heads=hq, n_kv_heads=hkv, d_ffn=f, vocab=v, dtype=dtype)
    w = synth.make_weights(cfg, 2115)
    kv = synth.make_kv_prefix(cfg, 2116, 16)
    t = [int(x) for x in synth.make_tokens(2117, most, v)]

    def run(n):
        def fn():
            g = gpu.GpuDrafter(cfg, w, max_batch=most, max_ctx=64, max_calib=1)
            try:
                g.set_groups(es.easyspec_default_groups(L, group, es.EASYSPEC_POLICY_ALIGNED))
                for b in range(n):
                    g.import_kv(b, *kv)
                return g.draft_step({b: t[b] for b in range(n)})[1][:n]
            finally:
                g.close()
        return both(monkeypatch, fn)

    for n, one_launch in ((1, True), (most, False)):
        a, b = run(n)
        assert np.array_equal(a, b) != one_launch, n
        gpu.assert_close(b, a, TOL[dtype], f"{n} columns")


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_against_the_oracle_batch(oracle, gpu, dtype):
    """Four sequences of unequal contexts drafting together, set sizes 1, 2, 1."""
    cfg = synth.model_shape("tiny", dtype=dtype)
    w = synth.make_weights(cfg, 2120)
    model = oracle.Model(cfg, w, 128)
    bounds = [0, 1, 3, 4]
    g = gpu.GpuDrafter(cfg, w, max_batch=4, max_ctx=128, max_calib=16)
    try:
        g.set_groups(bounds)
        seqs = []
        for b, n in enumerate((1, 13, 40, 97)):
            p = [int(x) for x in synth.make_tokens(2121 + b, n, cfg["vocab"])]
            seqs.append(oracle.Sequence(model))
            seqs[b].calibrate(p)
            g.prefill(b, p)
        for step in range(2):
            toks = {b: 7 * b + step for b in range(4)}
            _, lg = g.draft_step(toks)
            for b in range(4):
                gpu.assert_close(lg[b], seqs[b].fuzzy_step(bounds, toks[b]), TOL[dtype], f"step {step}, sequence {b}")
    finally:
        g.close()


def test_a_spoilt_token_reaches_no_earlier_row(gpu):
    cfg = synth.model_shape("tiny", dtype="bf16")
    w = synth.make_weights(cfg, 2130)
    bad, t = 77, [5, 9, 12, 77, 3, 8]

    def run():
        g = gpu.GpuDrafter(cfg, w, max_batch=1, max_ctx=64, max_calib=16)
        try:
            g.calibrate({0: [1, 2, 3]})
            return g.calibrate({0: t})[1][0]
        finally:
            g.close()

    clean = run()
    w["embed"] = w["embed"].copy()
    w["embed"][bad, 3] = 0x7FC0  # a bf16 NaN
    got = run()
    assert np.array_equal(got[:3], clean[:3]) and np.isnan(got[3:]).all()


def test_captured_and_replayed(gpu):
    """A captured pass replayed among eager passes of the same context, on a stream of its own."""
    import torch
    import paper_2502_02493_amd as es
    cfg = synth.model_shape("tiny")
    w = synth.make_weights(cfg, 2140)
    st = torch.cuda.Stream()
    g = gpu.GpuDrafter(cfg, w, max_batch=1, max_ctx=64, max_calib=16, stream=st.cuda_stream)
    try:
        with torch.cuda.stream(st):
            g.calibrate({0: [1, 2, 3, 4]})
            _, want = g.draft_step({0: 9})
            es.easyspec_truncate(g.ctx, 0, 4)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=st):
                es.easyspec_draft_step(g.ctx, g.tok_in, g.tok_out, g.logits)
            es.easyspec_truncate(g.ctx, 0, 4)
            for i in range(4):
                _, other = g.draft_step({0: 20 + i})  # other results in the same places
                assert not np.array_equal(other, want)
                es.easyspec_truncate(g.ctx, 0, 4)
                g.tok_in.fill_(9)
                graph.replay()
                st.synchronize()
                assert np.array_equal(g.logits.cpu().numpy(), want), i
    finally:
        g.close()


def test_two_contexts_at_once(gpu):
    """Passes of two contexts on two streams, enqueued without waiting: more workgroups than the device holds at once, and
    every value those of a context alone.  Their units wait only for units of their own pass that are done or being worked on."""
    import torch
    import paper_2502_02493_amd as es
    cfgs = [synth.model_shape("tiny_qwen", vocab=4000, dtype=dt) for dt in ("fp32", "bf16")]  # 256 workgroups of 95 KB of LDS each
    n_steps, gs = 24, []

    def steps(g, tok, out):
        es.easyspec_truncate(g.ctx, 0, 4)
        for i in range(n_steps):
            es.easyspec_draft_step(g.ctx, tok[i], g.tok_out, out[i])

    try:
        for i, cfg in enumerate(cfgs):
            st = torch.cuda.Stream()
            g = gpu.GpuDrafter(cfg, synth.make_weights(cfg, 2160 + i), max_batch=1, max_ctx=64, max_calib=16, stream=st.cuda_stream)
            tok = torch.from_numpy(synth.make_tokens(2170 + i, n_steps, cfg["vocab"]).reshape(n_steps, 1)).to(g.dev)
            gs.append((g, st, tok, [torch.zeros(n_steps, cfg["vocab"], device=g.dev) for _ in range(2)]))
            torch.cuda.synchronize()
            g.calibrate({0: [1, 2, 3, 4]})
            steps(g, tok, gs[-1][3][0])                                          # alone
            torch.cuda.synchronize()
        for _ in range(3):
            for g, _, tok, out in gs:
                steps(g, tok, out[1])                                            # both under way at the same time
        torch.cuda.synchronize()
        for g, _, _, (alone, together) in gs:
            assert np.isfinite(alone.cpu().numpy()).all() and torch.equal(alone, together)
            assert int(g.lens()[1][0]) == n_steps                                # no pass gave up
    finally:
        for g, *_ in gs:
            g.close()
