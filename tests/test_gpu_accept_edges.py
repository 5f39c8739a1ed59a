"""GPU parity of sampling acceptance where its kernels change shape: slices longer than a thread holds at once (8 slices of
more than 16 384 entries), the most positions (64: more (row, slice) terms than threads), masked vocabularies (minus
infinity logits, whole slices and whole threads of them), more chunk sums than the draw holds in LDS."""
import numpy as np
import pytest

from test_gpu_accept import es, make_case, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def compare(oracle, es, case, T):
    draft, dl, tl, r, u = case
    acc, bon = run_gpu(es, draft, dl, tl, r, u, T)
    checked = 0
    for b in range(draft.shape[0]):
        m, bonus, margin = oracle.accept(draft[b], dl[b], tl[b], r[b], u[b], T, with_margin=True)
        if margin > 1e-9:
            assert (int(acc[b]), int(bon[b])) == (m, bonus), (b, margin)
            checked += 1
    assert checked >= max(1, draft.shape[0] - 1)


@pytest.mark.parametrize("batch,gamma,V,noise", [(2, 3, 131073, 0.5), (2, 2, 152064, 0.4), (3, 64, 257, 0.05), (2, 1, 8, 1.0), (1, 1, 2100001, 0.3)])
def test_sizes(oracle, es, batch, gamma, V, noise):  # noqa: F811
    compare(oracle, es, make_case(2000 + V, batch, gamma, V, 0.8, noise), 0.8)


@pytest.mark.parametrize("V,keep", [(4099, slice(3000, 3100)), (4099, slice(0, 1)), (140001, slice(0, 140001, 17))])
def test_masked_vocabulary(oracle, es, V, keep):  # noqa: F811
    draft, dl, tl, r, u = make_case(2100 + V, 3, 4, V, 0.8, 0.4)
    mask = np.full(V, -np.inf, np.float32)
    mask[keep] = 0.0
    dl, tl = dl + mask, tl + mask
    draft[:] = np.argmax(dl, axis=-1)
    compare(oracle, es, (draft, dl, tl, r, u), 0.8)
