"""Device memory that a prior batch keeps: records for the workgroups there are, not for the most there can be."""
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
