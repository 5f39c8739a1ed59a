"""Draws of sampling acceptance whose threshold is a running sum itself: equal weights, as many in front of a gap of weightless
tokens as behind it, and u = 1/2.  The running sum stands at half of the total all through the gap, and there the kernel's sums of
neighbouring threads, added in different orders, differ in their last bits and rise and fall over the threshold.  Whatever
the rounding, the draw is the last token in front of the gap or the first one behind it, and the same at every call."""
import numpy as np
import pytest

from test_gpu_accept import es, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu

# (weights on each side, first token, gap): running sums of the kernel's order that cross the threshold more than once, or only
# at threads without a weight (12, 5, 100 and 84, 5, 100), found with a host model of that order
CASES = [(9, 1, 100), (12, 1, 30), (12, 5, 100), (14, 1, 100), (17, 5, 30), (18, 1, 30), (18, 5, 30), (24, 0, 30), (29, 17, 60),
         (42, 5, 30), (46, 5, 60), (49, 40, 100), (52, 1, 60), (83, 1, 60), (84, 5, 100), (100, 40, 30)]


def draw(es, cases, tokens_of, V):  # noqa: F811
    """One sequence per case, no drafted tokens: a draw from the target's own distribution."""
    n = len(cases)
    tl = np.full((n, 1, V), -np.inf, np.float32)
    want = []
    for i, (m, first, gap) in enumerate(cases):
        tok = tokens_of(np.r_[first:first + m, first + m + gap:first + 2 * m + gap])
        tl[i, 0, tok] = 0.0
        want.append((tok[m - 1], tok[m]))
    res = [run_gpu(es, np.zeros((n, 0), np.int32), np.zeros((n, 0, V), np.float32), tl, np.zeros((n, 0), np.float32),
                   np.full(n, 0.5, np.float32), 1.0)[1] for _ in range(3)]
    for got in res:
        for i in range(n):
            assert got[i] in want[i], (cases[i], got[i], want[i])
        assert np.array_equal(got, res[0])


def test_two_entries_a_thread(es):  # noqa: F811
    draw(es, CASES, lambda i: i, 300)


def test_eight_entries_a_thread(es):  # noqa: F811
    draw(es, CASES, lambda i: i // 2 * 8 + i % 2, 40960)


@pytest.mark.parametrize("case", CASES)
def test_across_chunks(es, case):  # noqa: F811
    """The same sums a chunk each instead of a thread each."""
    draw(es, [case], lambda i: i // 2 * 512 + i % 2, 150 * 512)
