"""bsse_solve_realised against the same procedure spelled out with bsse_eval, a sort and one
bsse_profile_lp (host, fp64) per profile: programs on the device -- one wavefront, four wavefronts, the
edge of what LDS holds -- and beyond it on the host; more profiles than may be solved, and fewer;
degenerate programs (duplicated columns, small integer payoffs).  The optimum is the same number: both
solvers take the same pivots."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make

pytestmark = pytest.mark.gpu


# (m, n, K, payoffs, storage, rows, most)
CASES = [(3, 3, 2, "normal", "f32", 2000, 1000), (16, 16, 4, "normal", "f32", 20000, 200), (8, 8, 4, "dup", "f32", 3001, 50),
         (8, 8, 8, "normal", "f32", 777, 1), (5, 2, 1, "normal", "f32", 300, 9), (12, 6, 3, "int", "f32", 5000, 100000),
         (16, 32, 8, "uniform", "bf16", 3000, 40), (30, 20, 12, "normal", "f32", 500, 30), (24, 24, 20, "normal", "f32", 100, 20),
         (40, 30, 16, "normal", "f32", 60, 20), (4, 1, 3, "normal", "f32", 100, 10), (6, 5, 3, "normal", "f32", 70000, 3)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "m%dn%dK%d%s%s_%d_%d" % c)
def test_realised_profiles(case):
    import torch
    m, n, K, kind, storage, count, most = case
    game = workloads.small_game(m, n, K, 31 + m + n, kind=kind, storage=storage)
    X = torch.from_numpy(workloads.host_candidates(m, count, 7, "dyadic" if kind == "dup" else "dirichlet")).cuda()
    with _make(game) as g:
        V = torch.empty(count, dtype=torch.float32, device="cuda")
        br = torch.empty((count, K), dtype=torch.int32, device="cuda")
        bsse.bsse_eval(g, X, count, V, br)
        Vh, brh = V.cpu().numpy(), br.cpu().numpy()
        order = np.argsort(-Vh, kind="stable")
        _, first = np.unique(brh[order], axis=0, return_index=True)
        heads = order[np.sort(first)]                    # most promising first
        for again in range(2):
            value, x, profile, n_profiles, n_solved = bsse.bsse_solve_realised(g, X, count, max_profiles=most)
            assert (n_profiles, n_solved) == (len(heads), min(len(heads), most))
            best = None
            for c in heads[:most]:
                ok, v, xv = bsse.bsse_profile_lp(game.A, game.B, game.prior, brh[c])
                if ok and (best is None or v > best[0]):
                    best = (v, xv, brh[c])
            assert value == best[0]
            assert np.array_equal(profile, best[2]) and np.array_equal(x, best[1].astype(np.float32))
