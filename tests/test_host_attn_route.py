"""Which attention kernel a pass of at most 16 columns takes, and with how many terms and tiles, from the library's own rule on
the host."""
import pytest

import easyspec_synth as synth
import paper_2502_02493_amd as es


def route(G, ctx, tok, n_set=1, **over):
    """Calibration of tok[b] tokens behind ctx[b] slots."""
    cfg = synth.model_shape("tiny", **{**dict(dtype="bf16", head_dim=128, n_q_heads=2 * G, n_kv_heads=2), **over})
    lens = [n + i + 1 for n, t in zip(ctx, tok) for i in range(t)]
    seqs = [b for b, t in enumerate(tok) for _ in range(t)]
    return es.easyspec_attention_route(es.make_config(cfg, 16, 65536, 16), lens, seqs, n_set)


VECTOR = (False, 0, 1)


@pytest.mark.parametrize("G,n,tiles", [(4, 3, 1), (4, 4, 1), (4, 5, 2), (4, 9, 4), (4, 16, 4), (7, 2, 1), (7, 3, 2), (8, 2, 1), (8, 5, 4)])
def test_query_rows(G, n, tiles):
    assert route(G, [254], [2]) == VECTOR                          # 256 slots: one piece
    assert route(G, [700], [1]) == VECTOR                          # a draft step
    assert route(G, [700], [n]) == (True, 3, tiles)
    assert route(G, [257 - n], [n]) == (True, 3, tiles)            # 257 slots
    assert route(G, [256 - n], [n]) == VECTOR
    assert route(G, [700], [-(-12 // G) - 1]) == VECTOR            # a column less than 12 rows


def test_much_work():
    assert route(4, [8192], [6]) == (True, 2, 2)
    assert route(4, [8192], [2], n_set=2) == (True, 2, 1)
    assert route(2, [8192], [6]) == (True, 2, 1)                   # no rule for short contexts with two heads per KV head
    assert route(2, [700], [6]) == VECTOR
    assert route(4, [700], [6], head_dim=64) == VECTOR
    assert route(4, [8192], [6], dtype="fp32") == VECTOR


@pytest.mark.parametrize("ctx,tok,mfma", [
    ([100, 16000], [3, 1], False), ([3000, 16000], [3, 1], False), ([1000, 6000], [3, 1], False), ([600, 2000], [3, 1], False),
    ([100, 100, 2000], [3, 3, 1], False), ([200, 200, 200, 2000], [4, 4, 4, 1], False), ([1000, 4000], [3, 2], False),
    ([2000, 600], [3, 1], True), ([2000, 2000], [3, 1], True), ([997, 2001], [4, 1], True), ([997, 2002], [4, 1], False),  # 1001 of 2002 slots: half
    ([1500] * 10, [3] + [1] * 9, True), ([500] * 5, [3, 2, 2, 2, 2], True),
])
def test_lone_columns_at_longer_contexts(ctx, tok, mfma):
    """Four heads per KV head: the sequence with the rows has at least half of the longest context.  Seven and eight: any does."""
    assert route(4, ctx, tok)[0] == mfma
    for G in (7, 8):
        assert route(G, ctx, tok)[0]


@pytest.mark.parametrize("ctx,tok,n_set", [([], [], 1), ([16], [17], 1), ([65536], [1], 1), ([16], [1], 0), ([16], [1], 9)])
def test_bad_arguments(ctx, tok, n_set):
    with pytest.raises(es.EasySpecError) as e:
        route(4, ctx, tok, n_set)
    assert e.value.code == es.EASYSPEC_EINVAL
