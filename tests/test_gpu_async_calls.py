"""bsse_eval and bsse_sweep_chunk do not wait for the device, on their first use and when their scratch
grows either."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make, _run_eval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def half_a_second():
    """Cycles of a kernel that spins for about that long."""
    import torch
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    start.record()
    torch.cuda._sleep(1_000_000)
    end.record()
    end.synchronize()
    return int(500.0 / start.elapsed_time(end) * 1_000_000)


@pytest.mark.parametrize("call", ["eval", "chunk"])
@pytest.mark.parametrize("shape", [(30, 50, 6, "f32"), (20, 2, 30, "f32"), (150, 9, 3, "f32"), (32, 32, 16, "f32"),
                                   (64, 128, 9, "bf16"), (8, 8, 4, "f32")], ids=lambda s: "m%dn%dK%d%s" % s)
def test_does_not_wait(shape, call, half_a_second):
    import torch
    m, n, K, storage = shape
    game = workloads.small_game(m, n, K, 5, kind="uniform" if storage == "bf16" else "normal", storage=storage)
    X = workloads.host_candidates(m, 9000, 3)
    with _make(game) as g:
        Xd, V, _ = _run_eval(g, X)
    with _make(game) as g:
        out = torch.zeros(9000, device="cuda")
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        bsse.bsse_set_stream(g, stream.cuda_stream)
        done = torch.cuda.Event()
        with torch.cuda.stream(stream):
            torch.cuda._sleep(half_a_second)
            done.record()
        for count in (100, 3000, 9000):                  # (the larger ones outgrow what the smaller ones use)
            if call == "eval":
                bsse.bsse_eval(g, Xd, count, out, None)
            else:
                bsse.bsse_sweep_chunk(g, Xd, count, 0)
        assert not done.query()
        best = int(np.argmax(V))
        if call == "chunk":
            res = bsse.bsse_sweep_result(g)
            assert (res.best_index, np.float32(res.best_value)) == (best, V[best])
        stream.synchronize()
        if call == "eval":
            assert np.array_equal(out.cpu().numpy(), V)
        bsse.bsse_set_stream(g, None)
