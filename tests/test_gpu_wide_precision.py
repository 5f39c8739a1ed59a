"""Precision of wide passes (bf16 calibrations of more than 16 columns) against a 64-bit evaluation: no further from it
than the passes of at most 16 columns that other calibrations run as, whose attention carries queries and probabilities in fp32
on these shapes (heads of 64 elements, or one or two query heads per KV head); and the same bits every time."""
import pytest

import easyspec_synth as synth

pytestmark = pytest.mark.gpu

SHAPE = dict(n_layers=1, d_model=1024, d_ffn=2048, vocab=2000, rms_eps=1e-6, rope_theta=10000.0, qkv_bias=0, dtype="bf16")
SEEDS = 8


# Every rounding of the path but the queries' and the probabilities' is common to both routes, and the median over rows
# leaves out the few rows that a flipped last bit of a cache entry dominates.  Queries in two terms (16 to 17 bits) in the wide
# pass put its median 7 % above (12 % on models twice as wide); with all 24 bits the two differ by at most 0.6 %, and
# the one- and two-at-a-time forms of the 16-column passes by 0.7 %.  Allowed: 2 %, three times that scatter.
@pytest.mark.parametrize("heads", [dict(n_q_heads=16, n_kv_heads=4, head_dim=64), dict(n_q_heads=16, n_kv_heads=16, head_dim=64),
                                   dict(n_q_heads=8, n_kv_heads=4, head_dim=128)])
def test_no_further_from_64_bits(monkeypatch, heads):
    import torch
    from perf import cases
    assert torch.cuda.is_available()
    monkeypatch.setitem(synth._SHAPES, "narrow", dict(SHAPE, **heads))
    case = cases._model("calib", "narrow", [100 + 13 * i for i in range(8)], tokens=9, all_rows=True)
    err = {None: [], "0": []}
    for seed in range(1, SEEDS + 1):
        st = cases.prepare(case, seed)
        want = cases.exact(case, seed)[0][:, :9]
        for env in err:
            if env is None:
                monkeypatch.delenv("EASYSPEC_PAIR_PASSES", raising=False)
            else:
                monkeypatch.setenv("EASYSPEC_PAIR_PASSES", env)
            got = cases.run(st)[0][:, :9].clone()
            err[env].append(((got.double() - want).norm(dim=-1) / want.norm(dim=-1)).flatten())
            assert torch.equal(got, cases.run(st)[0][:, :9]), "the same call twice"
    wide, narrow = (float(torch.cat(err[e]).median()) for e in (None, "0"))
    print(f"median row error: wide {wide:.3e}, passes of 16 columns {narrow:.3e}")
    assert wide < 1.02 * narrow
