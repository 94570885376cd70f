"""The short-row kernel at the edges of its row lengths, of its blocks of four actions and of its grids:
one workgroup, the ragged last one, several rounds, launches cut over the types; exact ties; every result
against the oracle, and one call against two chunks."""
import numpy as np
import pytest

from oracle import sweep as osweep
from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make

pytestmark = pytest.mark.gpu

# (m, n, K, storage): m * n <= 64 is where it is chosen
SHAPES = [(1, 1, 1, "f32"), (2, 31, 3, "f32"), (3, 3, 2, "f32"), (4, 15, 2, "bf16"), (5, 1, 70, "f32"), (6, 10, 3, "f32"), (7, 9, 5, "bf16"),
          (8, 7, 4, "f32"), (9, 7, 2, "f32"), (12, 5, 3, "bf16"), (13, 4, 3, "f32"), (16, 4, 33, "f32"), (20, 3, 130, "f32"), (24, 2, 2, "f32"),
          (23, 2, 4, "bf16")]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "m%dn%dK%d%s" % s)
@pytest.mark.parametrize("count", [1, 255, 257, 3001, 600011])
def test_short_rows_parity(shape, count):
    m, n, K, storage = shape
    if count == 600011 and m * n * K > 200:
        count = 70001
    game = workloads.small_game(m, n, K, 40 + m + n + K, kind="uniform" if storage == "bf16" else "normal", storage=storage)
    X = workloads.host_candidates(m, count, 3 + count, "dirichlet")
    _full_check(game, X, bsse.BSSE_PATH_AUTO, "valu")


@pytest.mark.parametrize("shape", [(3, 3, 2, "f32"), (5, 12, 3, "f32"), (9, 7, 40, "f32"), (20, 3, 6, "bf16")], ids=lambda s: "m%dn%dK%d%s" % s)
@pytest.mark.parametrize("count", [300, 20001])
def test_short_rows_exact_ties(shape, count):
    m, n, K, storage = shape
    game = workloads.small_game(m, n, K, 78, kind="dup", storage=storage)
    X = workloads.host_candidates(m, count, 79, "dyadic")
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "valu")
    assert rep.br_mismatch == 0
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0


@pytest.mark.parametrize("shape", [(3, 3, 2), (9, 7, 40)])
def test_one_call_and_chunks(shape):
    import torch
    m, n, K = shape
    game = workloads.small_game(m, n, K, 5)
    for count in (2, 513, 40000, 700001):
        X = torch.from_numpy(workloads.host_candidates(m, count, 6)).cuda()
        with _make(game) as g:
            whole = bsse.bsse_sweep(g, X, count)
            row = bsse.bsse_sweep_best_row(g)
            assert np.array_equal(row, X[whole.best_index].cpu().numpy())
            head = bsse.bsse_sweep(g, X[:count // 2], count // 2)
            bsse.bsse_sweep_chunk(g, X[count // 2:].clone(), count - count // 2, count // 2)
            out = bsse.bsse_sweep_result(g)
            assert head.n_evals == count // 2 * K
            assert (out.best_index, out.best_value, out.n_evals, out.n_tie_evals) == (whole.best_index, whole.best_value, whole.n_evals, whole.n_tie_evals)
            assert np.array_equal(out.best_response, whole.best_response) and np.array_equal(bsse.bsse_sweep_best_row(g), row)
