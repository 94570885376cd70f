"""Payoffs with a large part in common: the small part products decide most best responses, which are then
summed with all the others."""
import time

import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make, _run_eval, _torch

pytestmark = pytest.mark.gpu


def _offset_game(m, n, K, offset, types=slice(None)):
    game = workloads.small_game(m, n, K, 30 + m + n, "normal")
    game.B[types] += np.float32(offset)
    return game


# (every kernel by itself, and games on either side of the rule that chooses: 30 is near its line)
@pytest.mark.parametrize("m, n, K", [(32, 32, 1), (21, 32, 5), (32, 64, 3), (19, 64, 16)])
@pytest.mark.parametrize("offset", [30, 100, 1000])
@pytest.mark.parametrize("count", [33, 70001])
def test_parity(m, n, K, offset, count):
    X = workloads.host_candidates(m, count, 31 + count, "dirichlet")
    _full_check(_offset_game(m, n, K, offset), X, expect_path="mfma_split6")


@pytest.mark.parametrize("m, n", [(32, 32), (24, 64)])
def test_few_and_many_rows_and_ties_agree(m, n):
    """Whole launches, launches cut over the types, and columns that are equal."""
    game = _offset_game(m, n, 4, 300)
    game.B[:, :, n - 1] = game.B[:, :, 3]
    X = workloads.host_candidates(m, 66001, 32, "dirichlet")
    with _make(game) as g:
        _, V, br = _run_eval(g, X)
        for part in (slice(0, 33), slice(20000, 21000), slice(66000, 66001)):
            _, v, b = _run_eval(g, X[part])
            assert np.array_equal(v, V[part]) and np.array_equal(b, br[part])
    _full_check(game, X[:5000], expect_path="mfma_split6")


@pytest.mark.parametrize("n, most", [(32, 1.45), (64, 1.75)])
def test_time(n, most):
    """All products at once cost 1.2 (n = 32) and 1.45 (n = 64) of leaving the small ones out; leaving them out
    and summing most tiles again 1.67 and 2.2.  One type of sixteen with an offset leaves the game its filter: a
    sixteenth of that, 1.1 at most."""
    def best_time(offset, types=slice(None)):
        with _make(_offset_game(32, n, 16, offset, types)) as g:
            X = _torch().empty((1 << 20, 32), dtype=_torch().float32, device="cuda")
            bsse.bsse_dirichlet(g, 33, 0, 1 << 20, X)
            times = []
            for _ in range(30):
                start = time.perf_counter()
                bsse.bsse_sweep(g, X, 1 << 20)
                times.append(time.perf_counter() - start)
            return min(times)
    plain = best_time(0)
    assert best_time(1000) < most * plain
    assert best_time(1000, slice(0, 1)) < 1.3 * plain
