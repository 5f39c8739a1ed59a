"""GPU parity of calibrations and tree levels whose route the number of query rows decides (heads of 128, four or seven per KV
head): one column less and as many as the matrix-core kernel takes, one, two and four tiles of them, contexts that end as one piece
(256 slots) and one slot further, a second sequence with a single column."""
import numpy as np
import pytest

import easyspec_synth as synth
from test_gpu_attn_row_tiles import gpu  # noqa: F401
from test_gpu_nonfinite import run
from test_gpu_parity import iteration_parity
from test_gpu_tree import tree_parity

pytestmark = pytest.mark.gpu


def shape(G):
    return synth.model_shape("tiny", dtype="bf16", head_dim=128, n_q_heads=2 * G, n_kv_heads=2)


def route(cfg, context, n):
    import paper_2502_02493_amd as es
    return es.easyspec_attention_route(es.make_config(cfg, 2, 1024, 16), [context + i + 1 for i in range(n)] + [101], [0] * n + [1], 1)


@pytest.mark.parametrize("G,n", [(4, 2), (4, 3), (7, 1), (7, 2), (8, 2), (4, 8), (4, 15)])  # with the second sequence at most one pass
@pytest.mark.parametrize("context", [254, 321, 700])  # 254: 256 slots with two tokens, 257 with three
def test_calibration(gpu, monkeypatch, G, n, context):  # noqa: F811
    """Against the vector kernel, which the oracle tests pin: queries in two terms and probabilities of (at least) 24 bits on both.
    Both runs are the vector kernel's where the rule leaves the pass with it (a column less, one piece)."""
    cfg = shape(G)
    tiles = {1: 1, 2: 2}.get(-(-n * G // 16), 4)
    rows = n > 1 and n * G >= 12 and context + n > 256
    assert route(cfg, context, n) == ((True, 3, tiles) if rows else (False, 0, 1))
    w = synth.make_weights(cfg, 1400)
    toks = {0: [int(x) for x in synth.make_tokens(1401, n, cfg["vocab"])], 1: [5]}
    got, kv = run(gpu, cfg, w, [context, 100], toks)
    monkeypatch.setenv("EASYSPEC_ATTN_MFMA", "0")
    assert route(cfg, context, n) == (False, 0, 1)
    want, kv0 = run(gpu, cfg, w, [context, 100], toks)
    for b in toks:
        # sums in another order, products of 48 against 32 bits: 2^-22 an operation; a bf16 cache entry that rounds the other way
        # costs 2^-9 of one of some 300 slots, and few do
        rel = np.linalg.norm(got[b] - want[b]) / np.linalg.norm(want[b])
        assert rel < 2e-4, (b, rel)
        for x, y in zip(kv[b], kv0[b]):
            assert (x != y).mean() < 1e-3


@pytest.mark.parametrize("G", [4, 7])
def test_iteration(oracle, gpu, G):  # noqa: F811
    iteration_parity(oracle, gpu, shape(G), 1410, [0, 1, 3, 4], 300, 4, n_iters=1)


@pytest.mark.parametrize("G", [4, 7])
def test_tree(oracle, gpu, G):  # noqa: F811
    tree_parity(oracle, gpu, shape(G), 1420, [0, 1, 4], 270, [2, 3, 5])
