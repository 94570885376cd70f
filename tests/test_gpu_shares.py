"""Launches of the any-shape kernel cut into equal shares of (block of rows, types): shares that start and end
inside a block, that span several, one pair each, fewer pairs than workgroups; and the sizes at which it stays
uncut.  Against the oracle, and per-type outputs and values row by row against a launch over the same rows alone."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make, _run_eval

pytestmark = pytest.mark.gpu

# (m, n, K, storage): several tiles a type, one, two and four types a tile, types in several stages
SHAPES = [(16, 40, 7, "bf16"), (30, 50, 5, "f32"), (20, 20, 9, "f32"), (9, 13, 11, "f32"), (12, 7, 13, "bf16"),
          (100, 200, 2, "f32")]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "m%dn%dK%d%s" % s)
@pytest.mark.parametrize("count", [2, 300, 32769, 50001, 66001, 140001])
def test_shares_against_the_oracle(shape, count):
    m, n, K, storage = shape
    if m * n * K > 9000 and count > 33000:
        count = 25001
    game = workloads.small_game(m, n, K, 90 + m + n, kind="uniform" if storage == "bf16" else "normal", storage=storage)
    _full_check(game, workloads.host_candidates(m, count, 91), bsse.BSSE_PATH_AUTO, "mfma")


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "m%dn%dK%d%s" % s)
def test_every_row_whatever_its_share(shape):
    m, n, K, storage = shape
    game = workloads.small_game(m, n, K, 95 + m + n, kind="dup", storage=storage)
    X = workloads.host_candidates(m, 50001, 96)
    with _make(game) as g:
        _, V, br = _run_eval(g, X)
        for first, last in ((0, 1), (255, 258), (12000, 12400), (30000, 45000), (50000, 50001)):
            _, v, b = _run_eval(g, X[first:last])
            assert np.array_equal(v, V[first:last]) and np.array_equal(b, br[first:last])


@pytest.mark.parametrize("shape", [(30, 50, 2, "normal", "f32"), (20, 40, 3, "int", "f32"), (16, 40, 3, "uniform", "bf16"),
                                   (24, 20, 4, "normal", "f32"), (90, 33, 1, "uniform", "bf16")],
                         ids=lambda s: "m%dn%dK%d%s_%s" % s)
@pytest.mark.parametrize("count", [131072, 131073, 196609, 262401])
def test_more_blocks_than_two_a_compute_unit(shape, count):
    m, n, K, kind, storage = shape
    game = workloads.small_game(m, n, K, 97 + m + n, kind=kind, storage=storage)
    _full_check(game, workloads.host_candidates(m, count, 98), bsse.BSSE_PATH_AUTO, "mfma")
