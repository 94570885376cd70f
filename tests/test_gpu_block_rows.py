"""Generated rows of lengths that are not four times a power of two, by blocks in LDS: around the lengths
where the kernel changes, at the edges of a block of rows, in several sets and with a centre; every row
against the oracle's generator, and one call against two and against a misaligned output, bit for bit."""
import numpy as np
import pytest

from oracle import dirichlet as odir
from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [7, 9, 12, 30, 33, 100, 127, 250, 255, 257])
def test_block_rows(m):
    import torch
    rows = min(256, 8192 // m)                       # of one block
    seed, first = 91, (1 << 33) - 5
    centre = np.random.default_rng(m).dirichlet(np.ones(m)).astype(np.float32)
    with _make(workloads.small_game(m, 2, 1, seed=1)) as g:
        for count in (1, rows - 1, rows, rows + 1, 5 * rows + 3):
            buf = torch.zeros(count * m + 8, dtype=torch.float32, device="cuda")
            out = buf[:count * m].view(count, m)
            bsse.bsse_dirichlet(g, seed, first, count, out)
            got = out.cpu().numpy()
            assert np.allclose(got, odir.rows(seed, first, count, m), rtol=2e-6, atol=1e-9)
            assert float(buf[count * m:].abs().max()) == 0.0
            off = torch.empty(count * m + 1, dtype=torch.float32, device="cuda")[1:].view(count, m)
            cut = count // 2
            bsse.bsse_dirichlet(g, seed, first, cut, off[:cut])
            bsse.bsse_dirichlet(g, seed, first + cut, count - cut, off[cut:])
            assert np.array_equal(off.cpu().numpy().view(np.uint32), got.view(np.uint32))
            bsse.bsse_dirichlet_around(g, seed, first, count, centre, 0.25, out)
            around = np.float32(0.25) * got + np.float32(0.75) * centre
            assert np.array_equal(out.cpu().numpy().view(np.uint32), around.view(np.uint32))
