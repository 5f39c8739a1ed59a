"""The terms of sampling acceptance's statistics are exp((l - slice maximum) / T) as a division rounds the exponent, each
taken against the slice's own maximum: slices of two entries, whose sum 1 + exp(x / T) shows a single rounding more in x / T."""
import numpy as np
import pytest

from test_gpu_accept import es  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [0.8, 0.7, 1.1])
def test_terms_of_slices_of_two(es, T):  # noqa: F811
    import torch
    B, V = 4096, 16  # eight slices of two entries in the one target row of every sequence
    gen = torch.Generator(device="cuda").manual_seed(5)
    l = torch.zeros(B, V, device="cuda")
    l[:, 1::2] = -torch.empty(B, V // 2, device="cuda").uniform_(0.5, 2.0, generator=gen)
    u = torch.rand(B, device="cuda", generator=gen)
    bytes_ = es.easyspec_accept_workspace_bytes(B, 0, V)
    ws = torch.zeros(bytes_ // 8, dtype=torch.float64, device="cuda")
    acc, bonus = (torch.zeros(B, dtype=torch.int32, device="cuda") for _ in range(2))
    es.easyspec_accept(None, None, l, None, u, B, 0, V, T, acc, bonus, ws, torch.cuda.current_stream().cuda_stream)
    # a sequence's share of the workspace begins with (maximum, sum) of each of its row's eight slices
    stats = ws.view(B, -1)[:, :16].view(B, 8, 2)
    assert bool((stats[..., 0] == 0).all())
    # The same exponential of the same quotients: identical sums.  (Divided by a tensor: by a number, torch multiplies with its
    # reciprocal.)  With x * (1 / T) 6 % of the sums differ at T = 0.8, 0.7 % at 0.7.
    x = l[:, 1::2].double()
    want = 1.0 + torch.exp(x / torch.full_like(x, float(np.float32(T))))
    differ = float((stats[..., 1] != want).double().mean())
    assert differ == 0.0
