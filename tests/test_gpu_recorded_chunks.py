"""bsse_sweep_chunk recorded into a graph: a replay does what the call did, on the rows the buffer then
holds, whatever the handle has been used for in between; results and rows are those of the values that
bsse_eval gives."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make, _run_eval

pytestmark = pytest.mark.gpu

# (m, n, K, payoffs, storage)
GAMES = [(3, 3, 2, "normal", "f32"), (20, 2, 30, "normal", "f32"), (150, 9, 3, "normal", "f32"),
         (30, 50, 6, "normal", "f32"), (40, 40, 3, "normal", "f32"), (9, 7, 40, "dup", "f32"), (24, 40, 9, "uniform", "bf16"),
         (32, 32, 16, "normal", "f32"), (16, 16, 5, "dup", "f32"), (64, 128, 9, "uniform", "bf16"), (100, 256, 3, "int", "f32"),
         (8, 8, 4, "normal", "f32"), (8, 8, 12, "dup", "f32")]
N = 3001


class Recorder:
    """A handle on a stream of its own, sets of rows with their values, and the buffer graphs read."""

    def __init__(self, game):
        import torch
        m, n, K, kind, storage = game
        game = workloads.small_game(m, n, K, 70 + m + n + K, kind=kind, storage=storage)
        rows = "dyadic" if kind == "dup" else "dirichlet"
        self.host = [workloads.host_candidates(m, N, seed, rows) for seed in (1, 2, 3, 4)]
        with _make(game) as g:
            self.sets, self.V, self.br = zip(*(_run_eval(g, X) for X in self.host))
            self.ties = [bsse.bsse_sweep(g, X, N).n_tie_evals for X in self.sets]
        self.g = _make(game)
        self.X = self.sets[0].clone()
        self.stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        bsse.bsse_set_stream(self.g, self.stream.cuda_stream)

    def record(self, base):
        import torch
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=self.stream):
            bsse.bsse_sweep_chunk(self.g, self.X, N, base)
        return graph

    def replay(self, graph, s):
        import torch
        self.X.copy_(self.sets[s])
        torch.cuda.synchronize()
        with torch.cuda.stream(self.stream):
            graph.replay()

    def best(self, *parts):
        """(value, index, row, best responses, ties) over parts (set, index base)."""
        tops = []
        for s, base in parts:
            c = int(np.argmax(self.V[s]))
            tops.append((-float(self.V[s][c]), base + c, s, c))
        v, index, s, c = min(tops)
        return -v, index, self.host[s][c], self.br[s][c], sum(self.ties[s] for s, _ in parts)

    def check(self, out, *parts):
        v, index, row, br, ties = self.best(*parts)
        assert (out.best_value, out.best_index, out.n_tie_evals) == (v, index, ties)
        assert np.array_equal(out.best_response, br)
        self.check_row(*parts)

    def check_row(self, *parts):
        assert np.array_equal(bsse.bsse_sweep_best_row(self.g), self.best(*parts)[2])


@pytest.fixture
def recorder(request):
    r = Recorder(request.param)
    yield r
    bsse.bsse_set_stream(r.g, None)
    r.g.close()


_games = pytest.mark.parametrize("recorder", GAMES, indirect=True, ids=lambda s: "m%dn%dK%d%s%s" % s)


@_games
def test_replays_continue_the_sweep(recorder):
    r, g = recorder, recorder.g
    A, B, C, D = range(4)
    bsse.bsse_sweep_chunk(g, r.sets[A], N, 0)
    graph = r.record(N)
    r.replay(graph, B)
    r.check(bsse.bsse_sweep_result(g), (A, 0), (B, N))
    r.replay(graph, C)
    r.check_row((A, 0), (B, N), (C, N))                  # (the row is asked for while the replay runs)
    r.check(bsse.bsse_sweep_result(g), (A, 0), (B, N), (C, N))
    # a sweep in one call, then a replay
    r.check(bsse.bsse_sweep(g, r.sets[D], N), (D, 0))
    r.check(bsse.bsse_sweep_result(g), (D, 0))
    r.replay(graph, B)
    r.check(bsse.bsse_sweep_result(g), (D, 0), (B, N))
    bsse.bsse_sweep(g, r.sets[C], N)
    r.replay(graph, A)
    r.check_row((C, 0), (A, N))
    # the static scratch, another sweep, another replay
    r.check_row((C, 0), (A, N))
    v = r.best((D, 0))
    out = bsse.bsse_sweep_static(g, r.sets[D], N)
    assert (out.best_value, out.best_index, out.n_tie_evals) == (v[0], v[1], v[4])
    bsse.bsse_sweep_chunk(g, r.sets[B], N, 0)
    r.replay(graph, C)
    r.check(bsse.bsse_sweep_result(g), (B, 0), (C, N))


@_games
def test_a_recorded_first_chunk_starts_the_sweep_over(recorder):
    r, g = recorder, recorder.g
    A, B, C, D = range(4)
    r.check(bsse.bsse_sweep(g, r.sets[A], N), (A, 0))
    bsse.bsse_sweep_chunk(g, r.sets[A], N, 0)            # (the scratch that the graph names)
    bsse.bsse_sweep_reset(g)
    graph = r.record(0)
    for s in (B, C, D, B):
        r.replay(graph, s)
        r.check(bsse.bsse_sweep_result(g), (s, 0))
    bsse.bsse_sweep_chunk(g, r.sets[A], N, N)
    r.check(bsse.bsse_sweep_result(g), (B, 0), (A, N))
    bsse.bsse_sweep_reset(g)
    bsse.bsse_sweep_chunk(g, r.sets[A], 100, 0)
    bsse.bsse_sweep_result(g)
    r.replay(graph, C)
    bsse.bsse_sweep_chunk(g, r.sets[D], N, N)
    r.check(bsse.bsse_sweep_result(g), (C, 0), (D, N))


@_games
def test_recording_alone_changes_nothing(recorder):
    r, g = recorder, recorder.g
    A, B = 0, 1
    bsse.bsse_sweep_chunk(g, r.sets[A], N, 0)
    r.check(bsse.bsse_sweep(g, r.sets[B], N), (B, 0))
    graph = r.record(N)
    r.check(bsse.bsse_sweep_result(g), (B, 0))
    polished = bsse.bsse_polish(g)
    r.replay(graph, A)                                   # (polishing works on the result last reported)
    assert polished.value >= float(r.V[B].max()) and np.array_equal(bsse.bsse_polish(g).x, polished.x)
    r.check(bsse.bsse_sweep_result(g), (B, 0), (A, N))


@_games
def test_scratch_is_outgrown(recorder):
    """Larger chunks and generated sets after the recording: what the graph names stays as it was."""
    import torch
    r, g = recorder, recorder.g
    A, B = 0, 1
    bsse.bsse_sweep_chunk(g, r.sets[A], N, 0)
    graphs = [r.record(N)]
    big = torch.cat(list(r.sets) * 20)
    torch.cuda.synchronize()                             # (the rows are made on another stream than the handle's)
    for copies in (4, 20, 80):
        bsse.bsse_sweep_reset(g)
        bsse.bsse_sweep_chunk(g, big[:copies * N], copies * N, 0)
        bsse.bsse_sweep_result(g)
        graphs.append(r.record(N))
    for graph in graphs:
        bsse.bsse_sweep(g, r.sets[A], N)
        r.replay(graph, B)
        r.check(bsse.bsse_sweep_result(g), (A, 0), (B, N))
    # rows of the handle, then a set of another size
    bsse.bsse_dirichlet(g, 5, 0, N)
    rows = bsse.candidates_to_host(g)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=r.stream):
        bsse.bsse_sweep_chunk(g, None, 0, N)
    bsse.bsse_dirichlet(g, 6, 0, 40 * N)
    with torch.cuda.stream(r.stream):
        torch.full((40 * N, g.m), 7.0, device="cuda")    # (memory that was freed would hold these)
    bsse.bsse_sweep(g, r.sets[A], 1)
    with torch.cuda.stream(r.stream):
        graph.replay()
    out = bsse.bsse_sweep_result(g)
    first = bsse.bsse_sweep(g, r.sets[A], 1)
    second = bsse.bsse_sweep(g, torch.from_numpy(rows).cuda(), N)
    assert out.best_value == max(first.best_value, second.best_value)
    if second.best_value > first.best_value:
        assert out.best_index == N + second.best_index and np.array_equal(out.best_response, second.best_response)


@pytest.mark.parametrize("shape", [(150, 9, 3), (30, 50, 6), (32, 32, 16)], ids=lambda s: "m%dn%dK%d" % s)
def test_recording_needs_scratch(shape):
    import torch
    m, n, K = shape
    game = workloads.small_game(m, n, K, 3)
    with _make(game) as g:
        X = torch.from_numpy(workloads.host_candidates(m, N, 1)).cuda()
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        bsse.bsse_set_stream(g, stream.cuda_stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            X.add_(0.0)
            with pytest.raises(bsse.BsseError) as err:
                bsse.bsse_sweep_chunk(g, X, N, 0)
        assert err.value.status == bsse.BSSE_ESTATE
        graph.replay()                                   # (the capture itself is as good as before)
        torch.cuda.synchronize()
        bsse.bsse_set_stream(g, None)
