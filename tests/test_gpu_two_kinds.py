"""Any-shape games with a kernel for two workgroups a compute unit beside the one for three, and those whose
types take a long stage: the sizes between three and four blocks a compute unit, where the launch changes, and
recorded chunks that need more records than a greater one before them."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make, _run_eval, _torch

pytestmark = pytest.mark.gpu

# (m, n, K, payoffs, storage), rows in three blocks a compute unit.  K = 1 is never cut over the types.
SHAPES = [(70, 33, 1, "uniform", "bf16", 98304), (128, 20, 1, "uniform", "bf16", 98304), (100, 70, 1, "uniform", "bf16", 98304),
          (97, 38, 2, "uniform", "bf16", 98304), (120, 64, 1, "uniform", "bf16", 98304), (60, 40, 1, "normal", "f32", 98304),
          (40, 33, 1, "normal", "f32", 98304), (30, 50, 1, "normal", "f32", 196608), (20, 70, 1, "int", "f32", 196608)]
IDS = lambda s: "m%dn%dK%d%s_%s_%d" % s


def _make_game(shape, kind=None):
    m, n, K, payoffs, storage, _ = shape
    return workloads.small_game(m, n, K, 50 + m + n, kind or payoffs, storage)


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
@pytest.mark.parametrize("more", [0, 1, 32768, 32769])
def test_against_the_oracle(shape, more):
    count = shape[-1] + more * (shape[-1] // 98304)
    _full_check(_make_game(shape), workloads.host_candidates(shape[0], count, 51), expect_path="mfma")


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_rows_whatever_the_launch(shape):
    """The same bits in launches of every kind (exact ties among them)."""
    X = workloads.host_candidates(shape[0], shape[-1] + 20000, 52)
    with _make(_make_game(shape, "dup")) as g:
        _, V, br = _run_eval(g, X)
        for part in (slice(0, shape[-1]), slice(300, 30300), slice(5, 6)):
            _, v, b = _run_eval(g, X[part])
            assert np.array_equal(v, V[part]) and np.array_equal(b, br[part])


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_recorded_chunk_after_a_greater_one(shape):
    torch = _torch()
    m, count = shape[0], shape[-1]
    X = torch.from_numpy(workloads.host_candidates(m, count + 20000, 53)).cuda()
    with _make(_make_game(shape)) as g:
        expected = bsse.bsse_sweep(g, X, count)
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        bsse.bsse_set_stream(g, stream.cuda_stream)
        bsse.bsse_sweep_reset(g)
        bsse.bsse_sweep_chunk(g, X, count + 20000, 0)
        bsse.bsse_sweep_result(g)
        bsse.bsse_sweep_reset(g)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            bsse.bsse_sweep_chunk(g, X, count, 0)
        with torch.cuda.stream(stream):
            graph.replay()
        out = bsse.bsse_sweep_result(g)
        assert (out.best_index, out.best_value) == (expected.best_index, expected.best_value)
        bsse.bsse_set_stream(g, None)
