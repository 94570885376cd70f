"""The rules by which a game is given to a kernel with narrow operands, on the host."""
import numpy as np
import pytest

from paper_2605_18856_amd import workloads
from tests import kernels


def _wide(payoffs, m=100, K=2, seed=500):
    game = workloads.small_game(m, 256, K, seed, "int")
    game.B = np.random.default_rng(seed).integers(0, payoffs + 1, game.B.shape).astype(np.float32)
    return game


@pytest.mark.parametrize("forbidden", [-2.0 ** 20, -2.0 ** 54, -2.0 ** 57, -2.0 ** 60, 2.0 ** 100, -2.0 ** 120])
@pytest.mark.parametrize("payoffs", [1, 7])
def test_payoffs_that_a_large_one_hides(payoffs, forbidden):
    """Beside one action at +-2^57, what is left of 0 to 7 after taking off the middle of the range in 53 bits is one
    and the same number, which fits six bits."""
    game = _wide(payoffs)
    assert kernels.six_bit(game)
    game.B[1, 40, 17] = forbidden
    assert not kernels.six_bit(game)
    game.B[:, :, 17] = forbidden
    assert not kernels.six_bit(game)


@pytest.mark.parametrize("low, high, step, fits", [(0, 7, 1.0, True), (0, 15, 1.0, True), (-7, 7, 0.25, True), (100, 107, 1.0, True),
                                                   (-3, 12, 2.0 ** 40, True), (0, 16, 1.0, True), (0, 17, 1.0, False), (0, 100, 1.0, False)])
def test_spans_that_fit(low, high, step, fits):
    game = _wide(1)
    game.B = (step * np.random.default_rng(501).integers(low, high + 1, game.B.shape)).astype(np.float32)
    assert kernels.six_bit(game) == fits
