"""Games that the any-shape kernel sweeps in half-precision parts (m > 32, n > 16, fp32 payoffs that are no bf16
numbers): the edges of its k-steps and row tiles, ties and near ties, rows of any size, what the parts cannot hold, and
games that it leaves to the six products."""
import numpy as np
import pytest

from oracle import sweep as osweep
from paper_2605_18856_amd import bsse, workloads
from tests import kernels
from tests.test_gpu_parity import _full_check, _make, _run_eval

pytestmark = pytest.mark.gpu
IDS = lambda s: "m%dn%dK%d" % s


def _unseen(game, change):
    """change(type) for every type that the rule for half-precision parts does not sample (it takes eight evenly), so
    that the game keeps them."""
    assert game.K >= 16
    for t in range(1, game.K, 2):
        change(t)
    assert kernels.half_parts(game)
    return game


@pytest.mark.parametrize("shape", [(33, 17, 3), (48, 32, 2), (48, 33, 3), (49, 64, 2), (64, 65, 2), (65, 31, 2), (96, 97, 2),
                                   (97, 128, 2), (128, 20, 2), (128, 257, 1)], ids=IDS)
@pytest.mark.parametrize("kind", ["normal", "uniform"])
def test_edges(shape, kind):
    m, n, K = shape
    game = workloads.small_game(m, n, K, 300 + m + n, kind)
    assert kernels.half_parts(game)
    for count in (33, 4097):
        X = workloads.host_candidates(m, count, 301 + count, "dirichlet")
        rep, _ = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
        assert rep.br_mismatch == rep.flagged


@pytest.mark.parametrize("shape", [(40, 24, 16), (50, 90, 16), (100, 70, 16)], ids=IDS)
def test_exact_ties(shape):
    """Whole numbers of up to thirteen bits, a fifth of the columns twice (in every second type), dyadic rows: every sum
    is exact, so the ties and their number are the oracle's."""
    m, n, K = shape
    rng = np.random.default_rng(310 + m)
    game = workloads.small_game(m, n, K, 311, "normal")
    game.A = rng.integers(-4000, 4000, game.A.shape).astype(np.float32)
    game.B = rng.integers(-4000, 4000, game.B.shape).astype(np.float32)

    def twice(t):
        game.B[t, :, 1::5] = game.B[t, :, 0::5][:, :game.B[t, :, 1::5].shape[1]]
    _unseen(game, twice)
    for kind in ("dyadic", "vertex"):
        X = workloads.host_candidates(m, 2003, 312, kind)
        rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
        assert rep.br_mismatch == 0
        ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
        assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0


def _rounded_once(game, X):
    """Best responses on follower sums in 64 bits that are rounded to 32, by the rule: what the kernel's own sums must
    come to wherever they decide.  And how many evaluations tie."""
    best, ties = np.empty((len(X), game.K), np.int32), 0
    X = X.astype(np.float64)
    for t in range(game.K):
        u = (X @ game.B[t].astype(np.float64)).astype(np.float32)
        tied = u == u.max(axis=1, keepdims=True)
        best[:, t] = np.where(tied, X @ game.A[t].astype(np.float64), -np.inf).argmax(axis=1)
        ties += int((tied.sum(axis=1) > 1).sum())
    return best, ties


@pytest.mark.parametrize("shape", [(40, 24, 16), (64, 33, 16), (64, 90, 16), (96, 20, 16), (128, 70, 16), (128, 257, 16)], ids=IDS)
def test_ties_that_need_all_bits(shape):
    """Rows of multiples of 2^-12 and whole numbers of twelve or thirteen bits: all sums are exact, and ties hang on
    the product of the low parts (2049/4096 and 2047/4096 against (2049, 0) and (2, 2049))."""
    m, n, K = shape
    rng = np.random.default_rng(360 + m + n)
    game = workloads.small_game(m, n, K, 361, "normal")
    game.A = rng.integers(-4000, 4000, game.A.shape).astype(np.float32)
    game.B = rng.integers(-4000, -1999, game.B.shape).astype(np.float32)
    X = np.zeros((K * 40, m), np.float32)

    def pairs(t):
        i, k = rng.choice(m, 2, replace=False), 2 * int(rng.integers(1024, 1060)) + 1
        first, second, shift = rng.choice(n, 2, replace=False), rng.choice(n, 2, replace=False), 2 * int(rng.integers(40, 300))
        game.B[t, i] = -3999.0
        for pair in (first, second) if not set(first) & set(second) else (first,):
            game.B[t, i, pair[0]] = (4096 - k + shift, 0)
            game.B[t, i, pair[1]] = (shift, k)
        X[40 * t:40 * t + 40, i] = np.array([k, 4096 - k], np.float32) / 4096
    _unseen(game, pairs)
    rest = X.sum(axis=1) == 0
    X[rest] = workloads.host_candidates(m, int(rest.sum()), 362, "dyadic")
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    assert rep.br_mismatch == 0
    assert out.n_tie_evals == int((ref.gap == 0).sum()) >= 40 * (K // 2)


def _near_pairs(m, n, K):
    rng = np.random.default_rng(370 + m)
    game = workloads.small_game(m, n, K, 371 + m, "normal")

    def pairs(t):
        half = n // 2
        units = np.spacing(np.abs(game.B[t, :, :half])) * rng.integers(-2, 3, (m, half))
        game.B[t, :, half:2 * half] = game.B[t, :, :half] + units.astype(np.float32)
    return _unseen(game, pairs)


@pytest.mark.parametrize("shape", [(64, 24, 16), (64, 90, 16), (128, 257, 16)], ids=IDS)
def test_rows_alone_and_among_others(shape):
    """Two equal columns, and two more that tie with them in one row (by the product of low parts) and with each other in
    another: the first row has the same responses by itself, beside the other one and among many."""
    m, n, K = shape
    game = workloads.small_game(m, n, K, 375, "normal")
    rng = np.random.default_rng(376)
    game.B = rng.integers(-4000, -1999, game.B.shape).astype(np.float32)
    one, other = np.zeros((2, m), np.float32)
    one[:2], other[0] = (2049 / 4096, 2047 / 4096), 1.0

    def columns(t):
        game.B[t, :2, :] = -3999.0
        game.B[t, :2, 3:5] = [[2], [2049]]
        game.B[t, :2, n - 3:n - 1] = [[2049], [0]]
        game.A[t, :, n - 2] = 9.0
    _unseen(game, columns)
    rows = np.stack([one] * 3 + [other] * 3 + [one] * 64 + [other] * 64)
    with _make(game) as g:
        alone = _run_eval(g, one[None])[2][0]
        assert np.all(alone[1::2] == n - 2)
        for X in (np.stack([one, other]), np.stack([one, other] * 3), rows):
            br = _run_eval(g, X)[2]
            assert np.array_equal(br[X[:, 1] > 0], np.tile(alone, (int((X[:, 1] > 0).sum()), 1)))
    X = workloads.host_candidates(m, 4001, 373, "dirichlet")
    with _make(_near_pairs(m, n, K)) as g:
        br = _run_eval(g, X)[2]
        for c in range(0, len(X) - 3, 97):
            assert np.array_equal(_run_eval(g, X[c:c + 1])[2][0], br[c])
            assert np.array_equal(_run_eval(g, X[c:c + 3])[2], br[c:c + 3])


@pytest.mark.parametrize("shape", [(40, 24, 16), (60, 90, 16), (64, 33, 16), (96, 64, 16), (128, 257, 16)], ids=IDS)
@pytest.mark.parametrize("kind", ["sparse", "vertex", "dirichlet"])
def test_near_ties(shape, kind):
    """Pairs of columns a few last bits apart: the responses are those of the true sums, rounded once."""
    m, n, K = shape
    game = _near_pairs(m, n, K)
    X = workloads.host_candidates(m, 2003, 372, kind)
    best, ties = _rounded_once(game, X)
    with _make(game) as g:
        Xd, _, br = _run_eval(g, X)
        assert np.array_equal(br, best)
        assert bsse.bsse_sweep(g, Xd, len(X)).n_tie_evals == ties > 0


@pytest.mark.parametrize("shape", [(33, 17, 16), (45, 32, 16), (48, 64, 16), (47, 250, 16), (49, 33, 16), (62, 95, 16), (64, 128, 16),
                                   (66, 40, 16), (95, 200, 16), (97, 63, 16), (127, 31, 16), (128, 257, 16)], ids=IDS)
def test_single_columns(shape):
    """One to three rows a wavefront, which go one by one: rows that do not begin or end on a multiple of four, pairs in
    the first and the last row tile, rows below 2^-60."""
    m, n, K = shape
    game = _near_pairs(m, n, K)
    X = np.concatenate([workloads.host_candidates(m, 30, 390, kind) for kind in ("sparse", "dirichlet", "vertex")])
    X[40:50] = np.ldexp(X[40:50], -70)
    best = _rounded_once(game, np.where(X.max(axis=1, keepdims=True) < 2.0 ** -60, np.ldexp(X, 70), X))[0]
    with _make(game) as g:
        for c in range(0, len(X), 3):
            few = 1 + c % 2 + c % 4 // 2
            assert np.array_equal(_run_eval(g, X[c:c + few])[2], best[c:c + few]), c


@pytest.mark.parametrize("shape", [(40, 24, 2), (50, 90, 2), (128, 70, 1)], ids=IDS)
@pytest.mark.parametrize("small", [-12, -18, -24, -30])
def test_small_components_decide(shape, small):
    """Nearly all of a row on leader actions where every payoff is zero: the rest, 2^small of it, decides alone, and
    its bits below 2^-39 of the greatest component are not in the parts."""
    m, n, K = shape
    game = workloads.small_game(m, n, K, 320 + m, "normal")
    game.B[:, :m // 2] = 0.0
    assert kernels.half_parts(game)
    X = workloads.host_candidates(m, 3001, 321, "dirichlet").astype(np.float64)
    X[:, m // 2:] *= 2.0 ** small
    X = X.astype(np.float32)
    rep, _ = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
    assert rep.br_mismatch == rep.flagged


@pytest.mark.parametrize("shape", [(40, 24, 2), (60, 90, 2), (128, 70, 1)], ids=IDS)
def test_powers_of_two_change_nothing(shape):
    """Rows and payoffs times powers of two: the same best responses."""
    m, n, K = shape
    game = workloads.small_game(m, n, K, 330 + m, "normal")
    game.B = np.where(np.abs(game.B) < 2.0 ** -9, 0.0, game.B).astype(np.float32)
    X = workloads.host_candidates(m, 2011, 331, "dirichlet")
    X = np.where(X < 2.0 ** -14, 0.0, X).astype(np.float32)
    seen = []
    for rows, payoffs in ((0, 0), (40, 3), (59, 0), (70, -40), (-59, 0), (-75, -10), (0, -70), (0, 70)):
        g2 = workloads.small_game(m, n, K, 330 + m, "normal")
        g2.B = np.ldexp(game.B, payoffs).astype(np.float32)
        assert kernels.half_parts(g2)
        with _make(g2) as g:
            seen.append(_run_eval(g, np.ldexp(X, rows).astype(np.float32))[2])
    assert all(np.array_equal(seen[0], s) for s in seen[1:])


@pytest.mark.parametrize("shape", [(40, 24, 16), (64, 90, 16), (128, 257, 16)], ids=IDS)
def test_near_ties_of_rows_of_any_size(shape):
    """Sums within the margin and exact ties of rows times powers of two, down to subnormal numbers (rows are multiples of
    2^-9): as many ties, and the same responses while the leader's payoffs, which decide the ties, are no subnormal ones."""
    m, n, K = shape
    game = _near_pairs(m, n, K)
    game.B[1, :, 5] = game.B[1, :, 4]
    X = workloads.host_candidates(m, 1003, 381, "dirichlet")
    X = np.ldexp(np.round(np.ldexp(X, 9)), -9).astype(np.float32)
    with _make(game) as g:
        Xd, _, br = _run_eval(g, X)
        ties = bsse.bsse_sweep(g, Xd, len(X)).n_tie_evals
        assert ties > 0
        for power in (-140, -120, -100, -62, -58, 40, 62, 90, 110):
            Xd, _, scaled = _run_eval(g, np.ldexp(X, power).astype(np.float32))
            assert power < -110 or np.array_equal(br, scaled), power
            assert bsse.bsse_sweep(g, Xd, len(X)).n_tie_evals == ties, power


@pytest.mark.parametrize("shape", [(40, 24, 16), (64, 90, 16), (128, 257, 16)], ids=IDS)
def test_rows_and_types_of_zeros(shape):
    """Rows of zeros, types whose payoffs are all zero, and both at once: every action ties, the first one is reported
    where the leader's payoffs tie too."""
    m, n, K = shape
    game = workloads.small_game(m, n, K, 385, "normal")

    def zeros(t):
        game.B[t] = 0.0
    _unseen(game, zeros)
    X = workloads.host_candidates(m, 500, 386, "dirichlet")
    X[::3] = 0.0
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    assert rep.br_mismatch == 0 and out.n_tie_evals == int((ref.gap == 0).sum()) > 0


def test_whole_and_cut_launches_agree():
    game = workloads.small_game(50, 60, 16, 340, "normal")

    def twice(t):
        game.B[t, :, 59] = game.B[t, :, 58]
    _unseen(game, twice)
    X = workloads.host_candidates(50, 200003, 341, "dirichlet")
    with _make(game) as g:
        _, V, br = _run_eval(g, X)
        for part in (slice(0, 1), slice(1000, 1333), slice(190000, 200003)):
            _, v, b = _run_eval(g, X[part])
            assert np.array_equal(v, V[part]) and np.array_equal(b, br[part])


@pytest.mark.parametrize("why", ["forbidden", "whole", "rows_end"])
def test_what_the_parts_are_not_for(why):
    """Forbidden actions at -10^6 and whole numbers of 23 bits that are close to each other (six products), and rows of
    zeros (not)."""
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
    assert kernels.half_parts(game) == (why == "rows_end")
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
    if why != "forbidden":
        ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
        assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0
