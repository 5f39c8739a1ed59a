"""Sampling acceptance that gives up waiting for another workgroup's value (include/easyspec.h, easyspec_accept): -1, kernels that end,
and a workspace that serves the next call.  The give-up is forced from the host, which picks the kernel whose own bounded wait ends
before its first look."""
import numpy as np
import pytest

from test_gpu_accept import es, make_case  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,gamma,V", [(3, 4, 300), (2, 0, 512), (2, 5, 128256), (9, 5, 66001), (1, 1, 2100001)])
def test_give_up(oracle, es, batch, gamma, V):  # noqa: F811
    import torch
    draft, dl, tl, r, u = make_case(3300 + V, batch, gamma, V, 0.8, 0.5)
    dev = [torch.from_numpy(a).cuda() if a.size else None for a in (draft, dl, tl, r, u)]
    ws = torch.empty(es.easyspec_accept_workspace_bytes(batch, gamma, V) // 8, dtype=torch.float64, device="cuda")
    want = [oracle.accept(draft[b], dl[b], tl[b], r[b], u[b], 0.8, with_margin=True) for b in range(batch)]

    def call(fn):
        acc, bon = (torch.full((batch,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        fn(*dev, batch, gamma, V, 0.8, acc, bon, ws, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return list(zip(acc.tolist(), bon.tolist()))

    for _ in range(2):
        for b, got in enumerate(call(es.easyspec_accept_give_up)):
            if got != (-1, -1):  # all there at the first look: not with one chunk (512 entries), whose own sum is sent after it
                assert V > 512 and (got == want[b][:2] or want[b][2] <= 1e-9), (b, got)
        checked = 0
        for b, got in enumerate(call(es.easyspec_accept)):
            if want[b][2] > 1e-9:
                assert got == want[b][:2], b
                checked += 1
        assert checked >= max(1, batch - 1)
