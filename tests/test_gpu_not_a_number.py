"""Rows whose value is not a number, or minus infinity: every kernel reports minus infinity for them, their
neighbours keep their bits, no such row beats a number, and however a set of nothing else is swept the
answer is the same."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make, _run_eval

pytestmark = pytest.mark.gpu

# (m, n, K, payoffs, storage)
GAMES = [(3, 3, 2, "normal", "f32"), (20, 2, 30, "normal", "f32"), (150, 9, 3, "normal", "f32"),          # vector unit
         (9, 8, 5, "normal", "f32"), (20, 12, 3, "normal", "f32"), (40, 20, 3, "normal", "f32"),          # any shape
         (30, 50, 3, "normal", "f32"), (100, 70, 2, "normal", "f32"), (24, 7, 3, "uniform", "bf16"),
         (40, 90, 2, "uniform", "bf16"), (20, 40, 3, "int", "f32"),
         (32, 32, 4, "normal", "f32"), (16, 16, 5, "normal", "f32"), (100, 256, 3, "int", "f32"),         # listed shapes
         (64, 128, 4, "uniform", "bf16"), (16, 32, 3, "uniform", "bf16"), (8, 8, 4, "normal", "f32")]


def _sweeps(g, X):
    import torch
    Xd = torch.from_numpy(X).cuda()
    count, cut = len(X), len(X) // 3
    yield bsse.bsse_sweep(g, Xd, count)
    yield bsse.bsse_sweep_static(g, Xd, count)
    bsse.bsse_sweep_reset(g)
    bsse.bsse_sweep_chunk(g, Xd[:cut], cut, 0)
    bsse.bsse_sweep_chunk(g, Xd[cut:].clone(), count - cut, cut)
    yield bsse.bsse_sweep_result(g)


@pytest.mark.parametrize("game", GAMES, ids=lambda s: "m%dn%dK%d%s%s" % s)
@pytest.mark.parametrize("count", [300, 150001])
def test_rows_without_a_value(game, count):
    m, n, K, kind, storage = game
    game = workloads.small_game(m, n, K, 60 + m + n, kind=kind, storage=storage)
    game.A = game.A - np.float32(8.0)                    # every value is negative (still bf16 numbers where they were)
    if storage == "bf16":
        game.A = workloads.round_to_bf16(game.A)
    good = workloads.host_candidates(m, count, 9, "dirichlet")
    X = good.copy()
    bad = [0, 7, 31, 32, 100, count - 1]
    X[7] = np.nan
    for k, c in enumerate(bad):
        X[c, (k * 5) % m] = np.nan
    with _make(game) as g:
        _, V, br = _run_eval(g, X)
        _, want, want_br = _run_eval(g, good)
        assert np.all(np.isneginf(V[bad]))
        rest = np.setdiff1d(np.arange(count), bad)
        assert np.array_equal(V[rest], want[rest]) and np.array_equal(br[rest], want_br[rest])
        best = int(np.argmax(V))
        for out in _sweeps(g, X):
            assert (out.best_index, np.float32(out.best_value)) == (best, V[best])
            assert np.array_equal(out.best_response, br[best])
        priors = np.eye(K, dtype=np.float32)[:1]
        top = bsse.bsse_sweep_topk(g, 3, _run_eval(g, X)[0], count)
        assert top[1][0] == best and np.all(np.isfinite(top[0]))
        assert bsse.bsse_sweep_priors(g, priors, _run_eval(g, X)[0], count)[0].best_index not in bad
        X[:] = np.nan
        none = -1 if bsse.bsse_path_name(g).startswith("mfma_small") else 0
        for out in _sweeps(g, X):
            assert out.best_index == none and (none < 0 or np.isneginf(out.best_value))


@pytest.mark.parametrize("game", [g for g in GAMES if g[4] == "f32" and g[0] not in (3, 150)], ids=lambda s: "m%dn%dK%d%s%s" % s)
def test_sums_beyond_the_range(game):
    """Finite rows whose sums are all minus infinity: every action is a maximiser, and the value is what
    the vector unit makes of it."""
    m, n, K, kind, storage = game
    game = workloads.small_game(m, n, K, 61 + m + n, kind=kind, storage=storage)
    game.A = np.round(game.A) - np.float32(9.0)
    game.B = np.round(game.B) - np.float32(9.0)
    X = workloads.host_candidates(m, 500, 9, "dirichlet")
    X[::3] = np.float32(2.0 ** 126)
    with _make(game) as g, _make(game, bsse.BSSE_PATH_VALU) as v:
        Xd, V, br = _run_eval(g, X)
        _, want, want_br = _run_eval(v, X)
        assert np.all(np.isneginf(V[::3])) and np.all(np.isneginf(want[::3]))
        assert np.array_equal(br[::3], want_br[::3])
        best = int(np.argmax(V))
        for out in _sweeps(g, X):
            assert (out.best_index, np.float32(out.best_value)) == (best, V[best])
