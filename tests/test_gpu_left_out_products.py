"""Split operands whose small part products are left out where they decide nothing: rows where nothing but
them decides, ties, payoffs and rows of any size, and the launches that do and do not leave them out."""
import numpy as np
import pytest

from oracle import sweep as osweep
from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make, _run_eval

pytestmark = pytest.mark.gpu

# (m, n, K, payoffs): the listed shapes that leave products out, full and padded rows
SHAPES = [(32, 32, 3, "normal"), (20, 32, 2, "uniform"), (32, 64, 2, "normal"), (23, 64, 3, "normal"),
          (128, 256, 2, "int"), (100, 256, 1, "int")]
IDS = lambda s: "m%dn%dK%d%s" % s


def _paired_columns(game):
    """Every second column is its left neighbour but for the first four leader actions: high, high, low, low
    against low, low, high, high."""
    high, low = (7.0, 1.0) if np.all(game.B == np.round(game.B)) else (2.1, -1.9)
    game.B[:, :, 1::2] = game.B[:, :, 0::2]
    game.B[:, :2, 0::2], game.B[:, 2:4, 0::2] = high, low
    game.B[:, :2, 1::2], game.B[:, 2:4, 1::2] = low, high
    return game


def _near_equal_rows(m, count, seed):
    """Rows whose first four components are equal but for about 2^-16 of themselves: what decides between two
    paired columns is in the third bf16 parts of these."""
    rng = np.random.default_rng(seed)
    base = rng.uniform(0.1, 0.2, (count, 1))
    X = rng.dirichlet(np.ones(m), count) * (1 - 4 * base)
    X[:, :4] = base * (1 + np.ldexp(rng.standard_normal((count, 4)), -16))
    return X.astype(np.float32)


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
@pytest.mark.parametrize("count", [200, 66001])
def test_small_products_decide(shape, count):
    """Paired columns differ by what third parts weigh, which is more than 1e-6 of the sum's scale for most
    rows: those best responses have to be right.  (With a margin of nothing a hundred of 66001 rows are not.)"""
    m, n, K, kind = shape
    game = _paired_columns(workloads.small_game(m, n, K, 60 + m + n, kind))
    X = _near_equal_rows(m, count, 61)
    with _make(game) as g:
        assert bsse.bsse_path_name(g) == ("mfma_split3" if kind == "int" else "mfma_split6")
        Xd, V, br = _run_eval(g, X)
        out = bsse.bsse_sweep(g, Xd, count)
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    clear, close = ref.gap > 1e-6 * ref.scale, ref.gap < 2.0 ** -15 * ref.scale
    assert (clear & close).sum() > count // 4
    assert np.array_equal(br[clear], ref.br[clear])
    assert out.best_index == int(np.argmax(V)) and np.array_equal(out.best_response, br[out.best_index])


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
@pytest.mark.parametrize("rows, payoffs", [(1, 1), (-20, 0), (40, 3), (62, 0), (70, -40), (0, -60), (-45, -40), (0, 90)],
                         ids=lambda e: "2p%d" % e)
def test_powers_of_two_change_nothing(shape, rows, payoffs):
    """Rows and payoffs times powers of two: the same best responses, whatever the filter's norms and margins
    come to (beyond 2^64 the squares of a row overflow; rows below 2^-30 and payoffs below 2^-70 meet the least
    norm and margin)."""
    m, n, K, kind = shape
    game = workloads.small_game(m, n, K, 70 + m + n, kind)
    X = workloads.host_candidates(m, 20011, 71, "dirichlet")
    X = np.where(X < 2.0 ** -20, 0.0, X).astype(np.float32)
    game.B = np.where(np.abs(game.B) < 2.0 ** -9, 0.0, game.B).astype(np.float32)
    with _make(game) as g:
        _, _, br = _run_eval(g, X)
    game.B = np.ldexp(game.B, payoffs)
    with _make(game) as g:
        _, _, scaled = _run_eval(g, np.ldexp(X, rows))
    assert np.array_equal(br, scaled)


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_few_and_many_rows_agree(shape):
    """Launches cut over the types against whole ones, row by row, ties and near ties among them."""
    m, n, K, kind = shape
    game = _paired_columns(workloads.small_game(m, n, K, 80 + m + n, kind))
    game.B[:, :, n - 1] = game.B[:, :, n - 2]
    X = _near_equal_rows(m, 66001, 81)
    with _make(game) as g:
        _, V, br = _run_eval(g, X)
        for part in (slice(0, 33), slice(20000, 21000), slice(66000, 66001)):
            _, v, b = _run_eval(g, X[part])
            assert np.array_equal(v, V[part]) and np.array_equal(b, br[part])


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_infinite_sums_beside_near_ties(shape):
    """Rows whose sums are infinite have the same best responses among rows that are near a tie as by
    themselves (2^127 in one component: infinite where a payoff is 2 or more)."""
    m, n, K, kind = shape
    game = _paired_columns(workloads.small_game(m, n, K, 90 + m + n, kind))
    if kind == "uniform":
        game.B = (2.5 * game.B).astype(np.float32)
    X = _near_equal_rows(m, 66001, 91)
    big = np.zeros((66001, m), np.float32)
    big[np.arange(66001), 4 + np.arange(66001) % (m - 4)] = 2.0 ** 127
    among = np.arange(66001) % 7 == 3
    X[among] = big[among]
    with _make(game) as g:
        _, _, alone = _run_eval(g, big)
        _, _, br = _run_eval(g, X)
    assert np.array_equal(br[among], alone[among])
