"""GPU parity of sampling acceptance where its launches are cut differently: 8, 16, 32 and 64 slices of a row, two and eight
entries a thread, more chunks than the drawing workgroup has threads, ends of chunks, and a draw without a residual."""
import numpy as np
import pytest

from test_gpu_accept import es, make_case, run_gpu  # noqa: F401
from test_gpu_accept_edges import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,gamma,V", [
    (1, 5, 511), (1, 5, 512), (1, 5, 513),      # one chunk, a full one, one entry more
    (1, 5, 8192), (1, 5, 8193),                 # 16 chunks and one counter, 17 and two groups
    (1, 5, 16383), (1, 5, 16384),               # 8 slices, 16
    (1, 5, 32768), (1, 1, 65537),               # 32, 64
    (1, 31, 32769),                             # 16: four terms a thread
    (1, 5, 131072), (1, 5, 131073),             # 256 chunks, 257
    (9, 5, 66001),                              # 1161 chunks of two entries a thread: eight
    (5, 1, 300007),                             # slices longer than held, eight entries a thread
    (2, 20, 140003),                            # 41 rows: 16 slices longer than held
])
def test_cuts(oracle, es, batch, gamma, V):  # noqa: F811
    compare(oracle, es, make_case(3000 + V, batch, gamma, V, 0.9, 0.3), 0.9)


@pytest.mark.parametrize("V", [700, 140001])
@pytest.mark.parametrize("u", [0.0, 0.4])
def test_no_residual(oracle, es, V, u):  # noqa: F811
    draft, dl, tl, r, us = make_case(3100 + V, 2, 3, V, 0.8, 0.5)
    dl = tl[:, :3].copy()
    r[:] = 1.5  # rejects a pair of equal probabilities: the bonus is drawn from the target's own distribution
    us[:] = u
    compare(oracle, es, (draft, dl, tl, r, us), 0.8)


@pytest.mark.parametrize("V", [700, 140001])
def test_draw_at_the_total(es, V):  # noqa: F811
    draft, dl, tl, r, us = make_case(3200 + V, 2, 3, V, 0.8, 0.5)
    r[:], us[:] = 0.0, 1.0  # all accepted, u * sum is the sum: the last token with positive weight
    tl[:, 3, V - 300:] = -np.inf
    acc, bonus = run_gpu(es, draft, dl, tl, r, us, 0.8)
    assert acc.tolist() == [3, 3] and bonus.tolist() == [V - 301, V - 301]
