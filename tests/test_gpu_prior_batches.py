"""Prior batches: device memory for the workgroups there are, not for the most there can be; every number of types."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P, counts, most", [(65536, (1000,), 16 << 20), (65536, (1000, 70000), 96 << 20), (3, (1, 1 << 20), 64 << 20)])
def test_records_are_as_many_as_workgroups(P, counts, most):
    import torch
    game = workloads.small_game(4, 5, 2, 3)
    w = np.random.default_rng(1).random(P, dtype=np.float32)
    priors = np.stack([w, np.float32(1.0) - w], axis=1)
    with _make(game) as g:
        X = [torch.from_numpy(workloads.host_candidates(4, c, 2)).cuda() for c in counts]
        best = [bsse.bsse_sweep_priors(g, np.float32([[0.25, 0.75]]), x, len(x))[0] for x in X]
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for x, b in zip(X, best):
            priors[P // 2] = (0.25, 0.75)
            outs = bsse.bsse_sweep_priors(g, priors, x, len(x))
            assert (outs[P // 2].best_index, outs[P // 2].best_value) == (b.best_index, b.best_value)
        assert free - torch.cuda.mem_get_info()[0] <= most


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 8, 17])
@pytest.mark.parametrize("P, count", [(1, 1), (16, 4096), (17, 4097), (40, 100003)])
def test_every_number_of_types(K, P, count):
    """Bit for bit the sweep under each prior."""
    import torch
    game = workloads.small_game(5, 12, K, 30 + K)
    rng = np.random.default_rng(K)
    priors = rng.dirichlet(np.ones(K), size=P).astype(np.float32)
    priors[:, -1] += np.float32(1.0) - priors.sum(axis=1, dtype=np.float64).astype(np.float32)
    X = torch.from_numpy(workloads.host_candidates(5, count, 2)).cuda()
    with _make(game) as g:
        outs = bsse.bsse_sweep_priors(g, priors, X, count)
    for p in {0, P // 2, P - 1}:
        game.prior = priors[p]
        with _make(game) as g:
            one = bsse.bsse_sweep(g, X, count)
        assert (outs[p].best_index, outs[p].best_value) == (one.best_index, one.best_value)
        assert np.array_equal(outs[p].best_response, one.best_response)
