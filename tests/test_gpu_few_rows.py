"""Few rows on the general matrix-core kernel (a launch cut over the types, records folded on the host)
and ragged last tiles: the sweep in one call, streamed in two chunks, and through the static scratch
(never cut) agree bit for bit with the arg-max over bsse_eval's values, which the parity tests hold
against the oracle."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make

pytestmark = pytest.mark.gpu

# (m, n, K, payoffs, storage); the row counts reach from one row past the last size that is cut
GAMES = [(32, 32, 16, "normal", "f32"), (27, 32, 1, "normal", "f32"), (16, 16, 5, "dup", "f32"), (20, 64, 3, "normal", "f32"),
         (64, 128, 9, "uniform", "bf16"), (40, 128, 1, "uniform", "bf16"), (100, 256, 5, "int", "f32")]


@pytest.mark.parametrize("game", GAMES, ids=lambda s: "m%dn%dK%d%s%s" % s)
@pytest.mark.parametrize("count", [1, 33, 255, 257, 1000, 32769, 131072, 131073])
def test_few_rows(game, count):
    import torch
    m, n, K, kind, storage = game
    if count > 40000 and storage != "bf16":
        count = count // 4 + count % 2
    game = workloads.small_game(m, n, K, 900 + m + n + K, kind=kind, storage=storage)
    X = torch.from_numpy(workloads.host_candidates(m, count, 5 + count, "dyadic" if kind == "dup" else "dirichlet")).cuda()
    with _make(game) as g:
        V = torch.empty(count, dtype=torch.float32, device="cuda")
        br = torch.empty((count, K), dtype=torch.int32, device="cuda")
        bsse.bsse_eval(g, X, count, V, br)
        Vh = V.cpu().numpy()
        best = int(np.argmax(Vh))
        whole = bsse.bsse_sweep(g, X, count)
        row = bsse.bsse_sweep_best_row(g)
        cut = count // 3
        bsse.bsse_sweep_reset(g)
        if cut:
            bsse.bsse_sweep_chunk(g, X, cut, 0)
        bsse.bsse_sweep_chunk(g, X[cut:].clone(), count - cut, cut)
        early = bsse.bsse_sweep_best_row(g)
        parts = bsse.bsse_sweep_result(g)
        for out in (whole, parts, bsse.bsse_sweep_static(g, X, count)):
            assert (out.best_index, np.float32(out.best_value)) == (best, Vh[best])
            assert np.array_equal(out.best_response, br[best].cpu().numpy())
            assert (out.n_evals, out.n_tie_evals) == (count * K, whole.n_tie_evals)
        assert np.array_equal(row, X[best].cpu().numpy()) and np.array_equal(early, row)
        if kind == "dup" and count > 100:
            assert whole.n_tie_evals > 0
