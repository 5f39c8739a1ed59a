"""How many waves share a workgroup of a weight launch (host model of the launch; no GPU): launches that fill less than half of
the CUs take as many as leave each a single batch of loads if twelve are enough; larger ones and longer rows keep the
number that the operation takes everywhere else."""
import pytest

import easyspec_synth as synth
import paper_2502_02493_amd as es

QKV, O, GU, DOWN, HEAD = es.EASYSPEC_OP_QKV, es.EASYSPEC_OP_OPROJ, es.EASYSPEC_OP_GATEUP, es.EASYSPEC_OP_DOWN, es.EASYSPEC_OP_HEAD


def wide(d, dtype, vocab=32000):
    return synth.model_shape("tiny", dtype=dtype, d_model=d, d_ffn=4 * d, n_q_heads=d // 64, n_kv_heads=d // 256, vocab=vocab)


@pytest.mark.parametrize("cfg,op,waves", [
    (synth.model_shape("tiny_qwen"), QKV, 7), (synth.model_shape("tiny_qwen"), DOWN, 10), (synth.model_shape("tiny_qwen"), HEAD, 4),
    (synth.model_shape("tiny_qwen", dtype="bf16"), QKV, 4),
    (wide(768, "fp32"), QKV, 12), (wide(768, "fp32"), O, 6), (wide(1536, "bf16"), QKV, 12),   # the most
    (wide(512, "fp32"), DOWN, 8), (wide(1024, "fp32"), QKV, 8), (wide(1024, "bf16"), DOWN, 8),  # a single batch would take 16
    (wide(768, "fp32"), DOWN, 8), (wide(1536, "fp32"), QKV, 8), (wide(2048, "fp32"), DOWN, 8), (wide(2048, "fp32"), O, 8),  # more than 16
    (wide(2048, "fp32"), GU, 8),  # 512 workgroups
    (wide(2048, "fp32", 2000), HEAD, 8), (wide(4096, "bf16", 500), HEAD, 8), (wide(4096, "fp32"), HEAD, 4),  # few and many words
])
def test_waves(cfg, op, waves):
    rep = es.easyspec_weight_walk(es.make_config(cfg, 1, 64, 16), op, 1, 1)
    assert rep["waves"] == waves
    assert rep["missed_tiles"] == rep["repeated_tiles"] == rep["w_out_of_range"] == rep["x_out_of_range"] == 0
