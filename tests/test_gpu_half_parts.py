"""Games that the any-shape kernel sweeps in half-precision parts (m > 32, n > 16, fp32 payoffs that are no bf16
numbers): the edges of its k-steps and row tiles, ties, what the parts cannot hold, and games that it leaves to the
six products."""
import numpy as np
import pytest

from oracle import sweep as osweep
from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make, _run_eval

pytestmark = pytest.mark.gpu
IDS = lambda s: "m%dn%dK%d" % s


@pytest.mark.parametrize("shape", [(33, 17, 3), (48, 32, 2), (48, 33, 3), (49, 64, 2), (64, 65, 2), (65, 31, 2), (96, 97, 2),
                                   (97, 128, 2), (128, 20, 2), (128, 257, 1)], ids=IDS)
@pytest.mark.parametrize("kind", ["normal", "uniform"])
def test_edges(shape, kind):
    m, n, K = shape
    game = workloads.small_game(m, n, K, 300 + m + n, kind)
    for count in (33, 4097):
        X = workloads.host_candidates(m, count, 301 + count, "dirichlet")
        rep, _ = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
        assert rep.br_mismatch == rep.flagged


@pytest.mark.parametrize("shape", [(40, 24, 2), (50, 90, 2), (100, 70, 1)], ids=IDS)
def test_exact_ties(shape):
    """Whole numbers of up to thirteen bits, a fifth of the columns twice, dyadic rows: every sum is exact, so the
    ties and their number are the oracle's."""
    m, n, K = shape
    rng = np.random.default_rng(310 + m)
    game = workloads.small_game(m, n, K, 311, "normal")
    game.A = rng.integers(-4000, 4000, game.A.shape).astype(np.float32)
    game.B = rng.integers(-4000, 4000, game.B.shape).astype(np.float32)
    game.B[:, :, 1::5] = game.B[:, :, 0::5][:, :, :game.B[:, :, 1::5].shape[2]]
    for kind in ("dyadic", "vertex"):
        X = workloads.host_candidates(m, 5003, 312, kind)
        rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
        assert rep.br_mismatch == 0
        ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
        assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0


@pytest.mark.parametrize("shape", [(40, 24, 2), (50, 90, 2), (128, 70, 1)], ids=IDS)
@pytest.mark.parametrize("small", [-12, -18, -24, -30])
def test_small_components_decide(shape, small):
    """Nearly all of a row on leader actions where every payoff is zero: the rest, 2^small of it, decides alone, and
    its bits below 2^-39 of the greatest component are not in the parts."""
    m, n, K = shape
    game = workloads.small_game(m, n, K, 320 + m, "normal")
    game.B[:, :m // 2] = 0.0
    X = workloads.host_candidates(m, 3001, 321, "dirichlet").astype(np.float64)
    X[:, m // 2:] *= 2.0 ** small
    X = X.astype(np.float32)
    rep, _ = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
    assert rep.br_mismatch == rep.flagged


@pytest.mark.parametrize("shape", [(40, 24, 2), (60, 90, 2), (128, 70, 1)], ids=IDS)
def test_powers_of_two_change_nothing(shape):
    """Rows and payoffs times powers of two: the same best responses (rows beyond 2^60 and payoffs from 2^60 on are
    summed in six products)."""
    m, n, K = shape
    game = workloads.small_game(m, n, K, 330 + m, "normal")
    game.B = np.where(np.abs(game.B) < 2.0 ** -9, 0.0, game.B).astype(np.float32)
    X = workloads.host_candidates(m, 2011, 331, "dirichlet")
    X = np.where(X < 2.0 ** -14, 0.0, X).astype(np.float32)
    seen = []
    for rows, payoffs in ((0, 0), (40, 3), (59, 0), (70, -40), (-59, 0), (-75, -10), (0, -70), (0, 70)):
        g2 = workloads.small_game(m, n, K, 330 + m, "normal")
        g2.B = np.ldexp(game.B, payoffs).astype(np.float32)
        with _make(g2) as g:
            seen.append(_run_eval(g, np.ldexp(X, rows).astype(np.float32))[2])
    assert all(np.array_equal(seen[0], s) for s in seen[1:])


def test_whole_and_cut_launches_agree():
    game = workloads.small_game(50, 60, 6, 340, "normal")
    game.B[:, :, 59] = game.B[:, :, 58]
    X = workloads.host_candidates(50, 200003, 341, "dirichlet")
    with _make(game) as g:
        _, V, br = _run_eval(g, X)
        for part in (slice(0, 1), slice(1000, 1333), slice(190000, 200003)):
            _, v, b = _run_eval(g, X[part])
            assert np.array_equal(v, V[part]) and np.array_equal(b, br[part])


@pytest.mark.parametrize("why", ["forbidden", "whole", "rows_end"])
def test_what_the_parts_are_not_for(why):
    """Forbidden actions at -10^6, whole numbers of 23 bits (ties of sums that need them all), rows that end at zero."""
    m, n, K = 40, 50, 2
    game = workloads.small_game(m, n, K, 350, "normal")
    X = workloads.host_candidates(m, 3001, 351, "dirichlet")
    if why == "forbidden":
        game.B[:, :, ::4] = -1e6
    elif why == "whole":
        rng = np.random.default_rng(352)
        game.B = rng.integers(2 ** 22, 2 ** 22 + 3, game.B.shape).astype(np.float32)
        X = workloads.host_candidates(m, 3001, 353, "vertex")
    else:
        X[::3] = 0.0
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
    if why != "forbidden":
        ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
        assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0
