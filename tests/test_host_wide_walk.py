"""Host walk of the matrix products of wide passes (calibrations of more than 16 columns of bf16 models), through the index
functions that the kernel uses; no GPU: every (row tile, k-tile, column tile) is multiplied exactly once, every weight and
operand piece that is read lies inside its array and the last is reached, partial sums fit their buffer, and there is a kernel
for every cut that is chosen."""
import pytest

import easyspec_synth as synth
import paper_2502_02493_amd as es

OPS = {"QKV": es.EASYSPEC_OP_QKV, "O": es.EASYSPEC_OP_OPROJ, "GATEUP": es.EASYSPEC_OP_GATEUP, "DOWN": es.EASYSPEC_OP_DOWN,
       "HEAD": es.EASYSPEC_OP_HEAD}


def walk(shape, op, n_cols, **over):
    cfg = es.make_config(synth.model_shape(shape, dtype="bf16", **over), 16, 64, 16)
    r = es.easyspec_wide_walk(cfg, OPS[op], n_cols)
    what = (shape, over, op, n_cols, r)
    assert r["kernel"] == 1, what
    assert r["missed"] == r["repeated"] == r["misplaced"] == r["empty_splits"] == 0, what
    assert r["w_out_of_range"] == 0 and r["w_max"] == r["w_pieces"] - 1, what
    assert r["x_out_of_range"] == 0 and r["x_max"] == r["x_pieces"] - 1, what
    assert r["out_max"] < r["out_room"] if r["out_room"] else r["splits"] == 1, what
    return r


@pytest.mark.parametrize("shape,over", [("tiny", {}), ("tiny_qwen", {}), ("tiny", dict(vocab=1003, head_dim=128, n_q_heads=2, n_kv_heads=2)),
                                        ("tiny", dict(d_model=32 * 9, d_ffn=32 * 43, vocab=1))])
def test_small_shapes(shape, over):
    """Every column count; sizes that leave a last tile, a last stage and a last split that are not full."""
    for op in OPS:
        for n in range(17, 257):
            walk(shape, op, n, **over)


@pytest.mark.parametrize("shape", ["llama3_8b", "qwen2_7b"])
def test_large_shapes(shape):
    for op in OPS:
        for n in range(24, 257, 16) if op != "HEAD" else (24, 90, 250):
            walk(shape, op, n, vocab=20000)


@pytest.mark.parametrize("tile_rows", [8, 12, 14])
def test_tile_heights(monkeypatch, tile_rows):
    monkeypatch.setenv("EASYSPEC_TILE_ROWS", str(tile_rows))
    monkeypatch.setenv("EASYSPEC_QKV_TILE_ROWS", str(tile_rows & ~3))
    for op in ("QKV", "GATEUP"):
        for n in range(17, 257, 16):
            walk("tiny_qwen", op, n)


# The instantiations that the shipped shapes reach; the GPU tests of the wide pass run each of them.
@pytest.mark.parametrize("shape,op,n,row_tiles,col_tiles,col_blocks", [
    ("llama3_8b", "GATEUP", 24, 2, 2, 1), ("llama3_8b", "GATEUP", 40, 2, 3, 1), ("llama3_8b", "GATEUP", 64, 2, 4, 1),
    ("llama3_8b", "GATEUP", 80, 4, 3, 2), ("llama3_8b", "GATEUP", 128, 4, 4, 2), ("llama3_8b", "GATEUP", 256, 4, 8, 2),
    ("qwen2_7b", "GATEUP", 80, 4, 5, 1), ("qwen2_7b", "GATEUP", 96, 4, 6, 1), ("qwen2_7b", "GATEUP", 256, 4, 6, 3),
    ("llama3_8b", "DOWN", 130, 4, 5, 2), ("llama3_8b", "DOWN", 192, 4, 6, 2), ("llama3_8b", "DOWN", 256, 4, 8, 2),
])
def test_cuts(shape, op, n, row_tiles, col_tiles, col_blocks):
    r = walk(shape, op, n)
    assert (r["row_tiles"], r["col_tiles"], r["col_blocks"]) == (row_tiles, col_tiles, col_blocks)


def test_rejects_bad_arguments():
    cfg = es.make_config(synth.model_shape("tiny", dtype="bf16"), 16, 64, 16)
    fp32 = es.make_config(synth.model_shape("tiny", dtype="fp32"), 16, 64, 16)
    for args in ((cfg, OPS["QKV"], 16), (cfg, OPS["QKV"], 257), (cfg, es.EASYSPEC_OP_ATTN, 32), (fp32, OPS["QKV"], 32)):
        with pytest.raises(es.EasySpecError):
            es.easyspec_wide_walk(*args)
