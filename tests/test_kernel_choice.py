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


@pytest.mark.parametrize("change, fits", [(lambda B: B, True), (lambda B: B + 1000.0, False), (lambda B: np.where(np.arange(50) % 4, B, -1e6), False),
                                          (lambda B: np.repeat(B[:, :, ::2], 2, axis=2), False), (lambda B: B * 2.0 ** 101, False),
                                          (lambda B: np.round(B * 2.0 ** 22), True), (lambda B: 0.0 * B, False)],
                         ids=["as drawn", "in common", "forbidden", "twice", "large", "whole numbers", "zeros"])
def test_half_precision_parts(change, fits):
    """The rule for half-precision parts, which knows no scale: where six products are the faster ones (many values near
    the maximum) or the only ones (sums of ordinary rows may be infinite) they stay."""
    game = workloads.small_game(60, 50, 3, 510, "normal")
    game.B = change(game.B.astype(np.float64)).astype(np.float32)
    assert kernels.half_parts(game) == fits
    for power in (-20, -2, 2) if np.abs(game.B).max() < 2.0 ** 90 else ():
        game.B = np.ldexp(change(workloads.small_game(60, 50, 3, 510, "normal").B.astype(np.float64)), power).astype(np.float32)
        assert kernels.half_parts(game) == fits


@pytest.mark.parametrize("m, n, fits", [(32, 50, False), (33, 17, True), (33, 16, False), (128, 300, True), (129, 50, False)])
def test_shapes_of_half_precision_parts(m, n, fits):
    assert kernels.half_parts(workloads.small_game(m, n, 2, 511, "normal")) == fits
