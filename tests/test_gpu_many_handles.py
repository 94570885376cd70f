"""Several handles alive at once that share a kernel but not its launch: scratch in LDS of different sizes,
created in either order, used in turn and from threads, each on a stream of its own."""
import threading

import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make

pytestmark = pytest.mark.gpu

# groups of (m, n, K, payoffs, storage); the games of a group run on the same kernels
GROUPS = [[(30, 96, 4, "normal", "f32"), (32, 70, 3, "normal", "f32"), (20, 500, 2, "normal", "f32"), (17, 40, 9, "normal", "f32")],
          [(30, 150, 3, "uniform", "bf16"), (32, 40, 20, "uniform", "bf16"), (20, 130, 2, "uniform", "bf16")],
          [(128, 12, 5, "normal", "f32"), (100, 16, 1, "normal", "f32"), (97, 9, 30, "normal", "f32")],
          [(128, 30, 3, "normal", "f32"), (100, 20, 2, "normal", "f32")],
          [(100, 256, 1, "int", "f32"), (128, 256, 5, "int", "f32")],
          [(64, 128, 1, "uniform", "bf16"), (50, 128, 9, "uniform", "bf16")],
          [(20, 64, 1, "normal", "f32"), (32, 64, 7, "normal", "f32")]]


@pytest.mark.parametrize("group", GROUPS, ids=lambda s: "_".join("m%dn%dK%d" % x[:3] for x in s))
@pytest.mark.parametrize("order", [1, -1], ids=["as_listed", "reversed"])
def test_handles_side_by_side(group, order):
    import torch
    games = [workloads.small_game(m, n, K, 80 + m + n, kind=kind, storage=storage) for m, n, K, kind, storage in group[::order]]
    counts = [50, 3000, 70001]
    X = {g.m: torch.from_numpy(workloads.host_candidates(g.m, counts[-1], 4)).cuda() for g in games}

    def work(h, game):
        out = []
        for c in counts:
            s, (v, i, b) = bsse.bsse_sweep(h, X[game.m], c), bsse.bsse_sweep_topk(h, 2, X[game.m], c)
            out += [s.best_value, s.best_index, tuple(s.best_response), tuple(v), tuple(i), b.tobytes()]
        return out

    want = []
    for game in games:
        with _make(game) as h:
            want.append(work(h, game))
    handles = [_make(game) for game in games]
    for _ in range(2):
        assert [work(h, game) for h, game in zip(handles, games)] == want
    streams = [torch.cuda.Stream() for _ in games]
    torch.cuda.synchronize()
    for h, s in zip(handles, streams):
        bsse.bsse_set_stream(h, s.cuda_stream)
    got = [[] for _ in games]
    threads = [threading.Thread(target=lambda k=k: got[k].extend(work(handles[k], games[k]) for _ in range(5))) for k in range(len(games))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [[w] * 5 for w in want]
    for h in handles:
        h.close()
