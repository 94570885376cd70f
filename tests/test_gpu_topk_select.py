"""Selection by threshold where it can go wrong: around one workgroup's direct range and the block of 256
behind a head, k at both ends, and values in an order that makes many keys reach the first threshold
(ascending, descending, a few distinct values, all equal); the order is that of a stable sort of bsse_eval's
values."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["drawn", "ascending", "descending", "classes", "equal"])
@pytest.mark.parametrize("count", [1, 255, 257, 5000, 16384, 16385, 65537, 300001])
def test_topk_order(order, count):
    import torch
    m, n, K = (8, 8, 4) if count % 2 else (6, 5, 3)
    game = workloads.small_game(m, n, K, 17, kind="normal")
    X = torch.from_numpy(workloads.host_candidates(m, count, 11, "dirichlet")).cuda()
    with _make(game) as g:
        V = torch.empty(count, dtype=torch.float32, device="cuda")
        br = torch.empty((count, K), dtype=torch.int32, device="cuda")
        if order in ("ascending", "descending"):
            bsse.bsse_eval(g, X, count, V, None)
            X = X[torch.argsort(V, descending=order == "descending", stable=True)].contiguous()
        elif order == "classes":
            X = X[torch.arange(count, device="cuda") % min(count, 7)].contiguous()
        elif order == "equal":
            X = X[:1].repeat(count, 1).contiguous()
        bsse.bsse_eval(g, X, count, V, br)
        Vh, brh = V.cpu().numpy(), br.cpu().numpy()
        want = np.argsort(-Vh, kind="stable")
        for k in (1, 7, 64, 256):
            v, i, b = bsse.bsse_sweep_topk(g, k, X, count)
            w = want[:k]
            assert np.array_equal(i, w) and np.array_equal(v, Vh[w].astype(np.float64)) and np.array_equal(b, brh[w])
