"""Wide games with small whole-number payoffs (the six-bit matrix instruction) where that can go wrong: rows of every
padding, spans and middles of the payoffs, ties and near ties, rows of any size, whole and cut launches; and games of
the same shape whose payoffs do not fit."""
import numpy as np
import pytest

from oracle import sweep as osweep
from paper_2605_18856_amd import bsse, workloads
from tests import kernels
from tests.test_gpu_parity import _full_check, _make, _run_eval

pytestmark = pytest.mark.gpu
N = 256


def _game(m, K, low, high, seed, step=1.0):
    rng = np.random.default_rng(seed)
    game = workloads.small_game(m, N, K, seed, "int")
    game.B = (step * rng.integers(low, high + 1, game.B.shape)).astype(np.float32)
    game.A = rng.integers(-9, 10, game.A.shape).astype(np.float32)
    return game


@pytest.mark.parametrize("m", [3, 31, 64, 65, 97, 127, 128])
@pytest.mark.parametrize("count", [1, 129, 3001, 40001])
def test_rows_of_any_length(m, count):
    game = _game(m, 3 if count < 40000 else 1, 0, 7, 400 + m)
    assert kernels.six_bit(game)
    rep, _ = _full_check(game, workloads.host_candidates(m, count, 401, "dirichlet"), bsse.BSSE_PATH_AUTO, "mfma_split3")
    assert rep.br_mismatch == rep.flagged


@pytest.mark.parametrize("low, high, step", [(0, 1, 1.0), (0, 15, 1.0), (-7, 7, 0.25), (100, 107, 1.0), (-3, 12, 2.0 ** 40), (0, 16, 1.0),
                                             (0, 100, 1.0), (5, 5, 1.0)])
def test_spans_of_payoffs(low, high, step):
    """Spans up to sixteen steps fit (their middle is taken off), wider ones stay on bf16 parts, and so do equal payoffs,
    which tie."""
    game = _game(100, 2, low, high, 410 + high, step)
    assert kernels.six_bit(game) == (0 < high - low <= 16)
    rep, out = _full_check(game, workloads.host_candidates(100, 3001, 411, "dirichlet"), bsse.BSSE_PATH_AUTO, "mfma_split3")
    assert rep.br_mismatch == rep.flagged
    if low == high:
        assert out.n_tie_evals == 2 * 3001


@pytest.mark.parametrize("kind", ["dyadic", "vertex"])
def test_exact_ties(kind):
    game = _game(90, 3, 0, 7, 420)
    game.B[:, :, 1::8] = game.B[:, :, 0::8]
    assert kernels.six_bit(game)
    X = workloads.host_candidates(90, 2003, 421, kind)
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split3")
    assert rep.br_mismatch == 0
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0


@pytest.mark.parametrize("power", [-140, -100, -70, -30, 40, 70, 110])
def test_powers_of_two_change_nothing(power):
    game = _game(128, 2, 0, 7, 430)
    assert kernels.six_bit(game)
    X = workloads.host_candidates(128, 1003, 431, "dirichlet")
    X = np.where(X < 2.0 ** -9, 0.0, X).astype(np.float32)
    X = np.float32(2.0 ** -9) * np.round(X * 2.0 ** 9).astype(np.float32)       # (still exact as subnormal numbers)
    with _make(game) as g:
        _, _, br = _run_eval(g, X)
        _, _, scaled = _run_eval(g, np.ldexp(X, power).astype(np.float32))
    if power > -120:
        assert np.array_equal(br, scaled)
    else:                                                 # (sums of subnormal numbers may vanish; no fault, an action)
        assert np.all((scaled >= 0) & (scaled < N))


@pytest.mark.parametrize("rows, payoffs", [(-140, 0), (-60, -60), (0, -100), (120, -100), (127, -90), (100, 20)])
def test_rows_and_payoffs_of_any_size(rows, payoffs):
    """The same best responses and ties from rows of multiples of 2^-9 whatever the powers of two, also where rows beyond
    2^118 meet payoffs that are scaled up (the leader's payoffs are large enough not to become subnormal)."""
    game = _game(100, 2, 0, 7, 435)
    X = workloads.host_candidates(100, 1003, 436, "dirichlet")
    X = np.ldexp(np.round(np.ldexp(X, 9)), -9).astype(np.float32)
    if rows < -100:
        game.A = (2.0 ** 14 * np.clip(game.A, -3, 3)).astype(np.float32)
    elif rows > 110:
        game.A = (2.0 ** -14 * game.A).astype(np.float32)
    with _make(game) as g:
        Xd, _, br = _run_eval(g, X)
        ties = bsse.bsse_sweep(g, Xd, len(X)).n_tie_evals
    game.B = np.ldexp(game.B, payoffs).astype(np.float32)
    assert kernels.six_bit(game)
    with _make(game) as g:
        Xd, _, scaled = _run_eval(g, np.ldexp(X, rows).astype(np.float32))
        assert bsse.bsse_sweep(g, Xd, len(X)).n_tie_evals == ties > 0
    assert np.array_equal(br, scaled)


@pytest.mark.parametrize("spread", [0, 3, 6, 9])
@pytest.mark.parametrize("bits", [4, 6, 9])
def test_rows_with_exact_sums(spread, bits):
    """Rows of whole numbers of a few bits, blocks of 32 components up to 2^-spread smaller: with few bits two parts hold
    them and their sums tie exactly or not at all, with more they do not.  Equal columns in the types that the rule for
    the six-bit kernel does not sample."""
    m, K = 120, 16
    game = _game(m, K, 0, 7, 437)
    game.B[1::2, :, 1::4] = game.B[1::2, :, 0::4]
    assert kernels.six_bit(game)
    rng = np.random.default_rng(438 + spread + bits)
    X = rng.integers(0, 2 ** bits, (601, m)) * (rng.random((601, m)) < 0.3)
    X = X * np.repeat(np.ldexp(1.0, -rng.integers(0, spread + 1, (601, 4))), 32, axis=1)[:, :m]
    X = np.ldexp(X, -bits - 4).astype(np.float32)
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split3")
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    assert rep.br_mismatch == 0 and out.n_tie_evals == int((ref.gap == 0).sum()) > 601


def test_small_components_decide():
    """Nearly all of a row on leader actions where all payoffs are equal: the remainder decides."""
    game = _game(128, 2, 0, 7, 440)
    game.B[:, :64] = 3.0
    assert kernels.six_bit(game)
    for small in (-10, -17, -25):
        X = workloads.host_candidates(128, 2003, 441, "dirichlet").astype(np.float64)
        X[:, 64:] *= 2.0 ** small
        X[:, 32:48] *= 2.0 ** small
        rep, _ = _full_check(game, X.astype(np.float32), bsse.BSSE_PATH_AUTO, "mfma_split3")
        assert rep.br_mismatch == rep.flagged


def test_whole_and_cut_launches_agree():
    game = _game(128, 40, 0, 7, 450)
    game.B[:, :, 255] = game.B[:, :, 254]
    assert kernels.six_bit(game)
    X = workloads.host_candidates(128, 140001, 451, "dirichlet")
    with _make(game) as g:
        whole = bsse.bsse_sweep(g, *_device(X))
        _, V, br = _run_eval(g, X)
        assert (whole.best_index, np.float32(whole.best_value)) == (int(np.argmax(V)), V.max())
        assert np.array_equal(whole.best_response, br[whole.best_index])
        for part in (slice(0, 1), slice(1000, 1333), slice(100000, 107001)):
            _, v, b = _run_eval(g, X[part])
            assert np.array_equal(v, V[part]) and np.array_equal(b, br[part])


def _device(X):
    import torch
    return torch.from_numpy(X).cuda(), X.shape[0]


@pytest.mark.parametrize("forbidden", [-2.0 ** 57, -2.0 ** 60])
def test_small_payoffs_beside_a_large_one(forbidden):
    """Payoffs 0 to 7 and an action that nobody takes: the others are still told apart (by their own size, not by the
    large one's)."""
    game = _game(100, 2, 0, 7, 470)
    X = workloads.host_candidates(100, 3001, 471, "dirichlet")
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    game.B[:, :, 17] = forbidden
    with _make(game) as g:
        _, _, br = _run_eval(g, X)
    clear = (ref.gap > 1e-6 * ref.scale) & (ref.br != 17)
    assert clear.mean() > 0.9 and np.array_equal(br[clear], ref.br[clear])
    assert not kernels.six_bit(game)


def test_leader_payoffs_that_are_no_half_precision_numbers():
    """Those keep the bf16 parts of the general kernel."""
    game = _game(70, 2, 0, 7, 460)
    game.A[0, 0, 0] = 2.0 ** 17
    assert not kernels.six_bit(game)
    _full_check(game, workloads.host_candidates(70, 1001, 461, "dirichlet"), bsse.BSSE_PATH_AUTO, "mfma_split3")
