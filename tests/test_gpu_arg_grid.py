"""Every action of a row tile group as the unique maximiser, and every pair of two actions some distance apart
as a tie that the leader's payoff decides: whole numbers throughout, so the answers are exact."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make, _run_eval

pytestmark = pytest.mark.gpu

# (m, n, payoffs, storage): one, two, four and eight row tiles a type, rows of full length and shorter ones;
# then numbers of actions that are no whole row tiles, odd and even numbers of them
SHAPES = [(32, 32, "normal", "f32"), (30, 32, "int", "f32"), (16, 32, "normal", "bf16"), (32, 64, "normal", "f32"),
          (64, 128, "normal", "bf16"), (50, 128, "normal", "bf16"), (128, 256, "int", "f32"),
          (20, 20, "normal", "f32"), (9, 31, "normal", "bf16"), (30, 50, "normal", "f32"), (40, 33, "int", "f32"),
          (50, 100, "normal", "bf16"), (100, 200, "int", "f32"), (16, 65, "normal", "bf16"), (8, 129, "normal", "f32")]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "m%dn%d%s_%s" % s)
@pytest.mark.parametrize("apart", [0, 1, 4, 8, 16, 32, 36])
@pytest.mark.parametrize("count", [45, 33000])
def test_every_action_and_every_pair(shape, apart, count):
    m, n, kind, storage = shape
    K = n
    game = workloads.small_game(m, n, K, 10 * n + m, kind, storage)
    rng = np.random.default_rng(11 * n + apart)
    t = np.arange(K)
    other = (t + apart) % n
    low, one = (0.0, 1.0) if kind == "int" else (-0.3125, 1.0 + 2.0 ** -7)        # (the second: no whole numbers)
    game.B = np.full((K, m, n), low, np.float32)
    game.B[t, :, t] = game.B[t, :, other] = one
    game.A = rng.integers(-4, 5, (K, m, n)).astype(np.float32)
    X = rng.integers(0, 4, (count, m)).astype(np.float32) / 8
    X[:, 0] += 0.125
    first, second = X @ game.A[t, :, t].T, X @ game.A[t, :, other].T
    low_action = np.minimum(t, other)
    want = np.where(first > second, t, np.where(second > first, other, low_action))
    with _make(game) as g:
        _, _, br = _run_eval(g, X)
    assert np.array_equal(br, want)
