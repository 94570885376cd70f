"""Evaluations of few rows recorded into a graph, on a handle that has no scratch yet and on one whose
scratch a later call outgrows: nothing is allocated or waited for, and every replay gives what the calls
give outside it."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fresh", [True, False], ids=["fresh", "used"])
@pytest.mark.parametrize("shape", [(30, 50, 6, "f32"), (9, 7, 40, "f32"), (32, 32, 16, "f32"), (64, 128, 9, "bf16"), (8, 8, 4, "f32")],
                         ids=lambda s: "m%dn%dK%d%s" % s)
def test_recorded_eval(shape, fresh):
    import torch
    m, n, K, storage = shape
    count = 1000
    game = workloads.small_game(m, n, K, 21, kind="normal", storage=storage)
    sets = [torch.from_numpy(workloads.host_candidates(m, count, seed)).cuda() for seed in (1, 2, 3)]
    want = []
    with _make(game) as g:
        for X in sets:
            V, br = torch.empty(count, device="cuda"), torch.empty((count, K), dtype=torch.int32, device="cuda")
            bsse.bsse_eval(g, X, count, V, br)
            want.append((V.cpu().numpy(), br.cpu().numpy()))
    with _make(game) as g:
        X = sets[0].clone()
        V, br = torch.zeros(count, device="cuda"), torch.zeros((count, K), dtype=torch.int32, device="cuda")
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        bsse.bsse_set_stream(g, stream.cuda_stream)
        if not fresh:
            bsse.bsse_eval(g, X, count, V, br)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            bsse.bsse_eval(g, X, count, V, br)
        if not fresh:                                # (scratch of three times the size from here on)
            big, Vb = torch.cat(sets), torch.empty(3 * count, device="cuda")
            torch.cuda.synchronize()
            bsse.bsse_eval(g, big, 3 * count, Vb, None)
            torch.cuda.synchronize()
            assert np.array_equal(Vb.cpu().numpy(), np.concatenate([w[0] for w in want]))
        for i in (0, 1, 2, 0):
            X.copy_(sets[i])
            V.zero_()
            br.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(V.cpu().numpy(), want[i][0]) and np.array_equal(br.cpu().numpy(), want[i][1])
        bsse.bsse_set_stream(g, None)
