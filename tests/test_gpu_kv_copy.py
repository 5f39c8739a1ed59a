"""KV import and export on device arrays (the copy kernel works on the caller's own memory), on host arrays and on
device arrays at addresses that do not suit 16-byte accesses (both through a staging array): every byte arrives, no
other sequence's slots and nothing past the imported slots is touched."""
import numpy as np
import pytest

import easyspec_synth as synth

pytestmark = pytest.mark.gpu


# a workgroup moves 2048 16-byte pieces of one (layer, KV head)'s run: 8 pieces a slot (bf16, 64-element heads), 16 (fp32)
@pytest.mark.parametrize("dtype,n", [("bf16", 1), ("bf16", 255), ("bf16", 256), ("bf16", 257), ("fp32", 127), ("fp32", 128), ("fp32", 300)])
def test_device_host_and_odd_addresses(dtype, n):
    import torch
    import paper_2502_02493_amd as es
    assert torch.cuda.is_available()
    cfg = synth.model_shape("tiny", dtype=dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    shape = (cfg["n_layers"], cfg["n_kv_heads"], n, cfg["head_dim"])
    gen = torch.Generator(device="cuda").manual_seed(n)
    ctx = es.easyspec_create(es.make_config(cfg, 3, 304, 4), torch.cuda.current_stream().cuda_stream)
    try:
        full = (cfg["n_layers"], cfg["n_kv_heads"], 304, cfg["head_dim"])
        held = {b: [torch.randn(full, generator=gen, device="cuda").to(dt) for _ in range(2)] for b in range(3)}
        for b in held:
            es.easyspec_kv_import(ctx, b, held[b][0], held[b][1], 304)

        def export(b):
            out = [torch.zeros(full, dtype=dt, device="cuda") for _ in range(2)]
            es.easyspec_kv_export(ctx, b, out[0], out[1], 304)
            return out

        new = [torch.randn(shape, generator=gen, device="cuda").to(dt) for _ in range(2)]

        def check(what):
            for x, y in zip(held[1], new):
                x[:, :, :n] = y
            for b in held:
                for x, y in zip(export(b), held[b]):
                    assert torch.equal(x, y), (what, b)

        es.easyspec_kv_import(ctx, 1, new[0], new[1], n)
        check("device")
        host = [torch.randn(shape, generator=gen, device="cuda").to(dt) for _ in range(2)]
        new = host
        as_np = [h.cpu().view(torch.int16 if dtype == "bf16" else torch.int32).numpy() for h in host]
        es.easyspec_kv_import(ctx, 1, as_np[0], as_np[1], n)
        check("host")
        new = [torch.randn(shape, generator=gen, device="cuda").to(dt) for _ in range(2)]
        odd = []
        for x in new:
            buf = torch.zeros(x.numel() + 1, dtype=dt, device="cuda")  # the view starts one element past a 16-byte boundary
            buf[1:].copy_(x.reshape(-1))
            odd.append(buf[1:])
        es.easyspec_kv_import(ctx, 1, odd[0], odd[1], n)
        check("odd address")
        # export: device, host and an odd address agree; nothing is written past the array
        want = [x[:, :, :n].contiguous() for x in held[1]]
        back_np = [np.zeros_like(a) for a in as_np]
        es.easyspec_kv_export(ctx, 1, back_np[0], back_np[1], n)
        for x, y in zip(back_np, want):
            assert np.array_equal(x, y.cpu().view(torch.int16 if dtype == "bf16" else torch.int32).numpy())
        for first in (0, 1):
            bufs = [torch.full((want[0].numel() + 16,), 7.0, dtype=dt, device="cuda") for _ in range(2)]
            es.easyspec_kv_export(ctx, 1, *[x[first:first + want[0].numel()] for x in bufs], n)
            for x, y in zip(bufs, want):
                assert torch.equal(x[first:first + y.numel()].view(y.shape), y)
                assert bool((x[:first] == 7).all()) and bool((x[first + y.numel():] == 7).all())
        same = torch.zeros_like(want[0])                     # one array for both: K, then V over it
        es.easyspec_kv_export(ctx, 1, same, same, n)
        assert torch.equal(same, want[1])
    finally:
        es.easyspec_destroy(ctx)
