"""The any-shape matrix-core kernel at the sizes where it can go wrong: edges of the row tiles, of the
k-steps and of the forms (types per tile, one tile per type, several), types that do not fit one LDS
stage, ragged and tiny batches (type-sliced launches), exact ties; every result against the oracle."""
import numpy as np
import pytest

from oracle import sweep as osweep
from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make

pytestmark = pytest.mark.gpu

# (m, n, K, storage)
SHAPES = [
    (9, 8, 5, "f32"), (33, 3, 6, "f32"), (128, 5, 3, "f32"), (17, 7, 4, "bf16"), (100, 8, 9, "bf16"),
    (8, 9, 3, "f32"), (16, 15, 2, "f32"), (48, 16, 5, "f32"), (65, 12, 1, "f32"), (20, 16, 7, "bf16"),
    (4, 17, 3, "f32"), (30, 31, 4, "f32"), (33, 32, 2, "f32"), (64, 20, 3, "f32"), (128, 29, 2, "f32"),
    (32, 32, 5, "bf16"), (70, 18, 3, "bf16"),
    (2, 33, 4, "f32"), (17, 50, 3, "f32"), (32, 65, 2, "f32"), (47, 96, 3, "f32"), (96, 40, 2, "f32"),
    (128, 100, 2, "f32"), (127, 255, 1, "f32"), (3, 300, 2, "f32"),
    (50, 100, 3, "bf16"), (64, 127, 2, "bf16"), (112, 260, 2, "bf16"), (16, 64, 3, "bf16"), (128, 256, 2, "bf16"),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "m%dn%dK%d%s" % s)
@pytest.mark.parametrize("count", [1, 129, 3001, 70001])
def test_any_shape_parity(shape, count):
    m, n, K, storage = shape
    if count == 70001 and m * n * K > 30000:
        count = 20011
    game = workloads.small_game(m, n, K, 40 + m + n + K, kind="uniform" if storage == "bf16" else "normal",
                                storage=storage)
    X = workloads.host_candidates(m, count, 3 + count, "dirichlet")
    _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_bf16" if storage == "bf16" else "mfma_split6")


@pytest.mark.parametrize("shape", [(9, 8, 5, "f32"), (20, 13, 3, "f32"), (20, 30, 3, "f32"), (40, 90, 2, "f32"),
                                   (100, 200, 2, "f32"), (24, 7, 3, "bf16"), (40, 90, 2, "bf16")],
                         ids=lambda s: "m%dn%dK%d%s" % s)
@pytest.mark.parametrize("kind", ["dyadic", "vertex"])
def test_any_shape_exact_ties(shape, kind):
    """Integer payoffs, duplicated follower columns, exactly representable candidates: every sum is
    exact, so the ties and their count are the oracle's."""
    m, n, K, storage = shape
    game = workloads.small_game(m, n, K, 78, kind="dup", storage=storage)
    for count in (300, 40000 if m * n < 2000 else 9000):
        X = workloads.host_candidates(m, count, 79, kind)
        rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_bf16" if storage == "bf16" else "mfma_split3")
        assert rep.br_mismatch == 0
        ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
        assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0


def test_one_call_and_streamed_sweeps_agree_and_continue():
    """One call leaves its result on the host; a chunk submitted afterwards continues that sweep."""
    import torch
    game = workloads.small_game(30, 50, 6, 5)
    count = 30011
    X = torch.from_numpy(workloads.host_candidates(30, count, 6)).cuda()
    with _make(game) as g:
        whole = bsse.bsse_sweep(g, X, count)
        row = bsse.bsse_sweep_best_row(g)
        assert np.array_equal(row, X[whole.best_index].cpu().numpy())
        for cut in (1, 300, 20000):
            head = bsse.bsse_sweep(g, X[:cut], cut)
            assert np.array_equal(bsse.bsse_sweep_best_row(g), X[head.best_index].cpu().numpy())
            bsse.bsse_sweep_chunk(g, X[cut:].clone(), count - cut, cut)
            out = bsse.bsse_sweep_result(g)
            assert (out.best_index, out.best_value, out.n_evals) == (whole.best_index, whole.best_value, whole.n_evals)
            assert np.array_equal(out.best_response, whole.best_response)
            assert np.array_equal(bsse.bsse_sweep_best_row(g), row)
