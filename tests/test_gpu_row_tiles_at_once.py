"""Types of two to four row tiles on the any-shape kernel (32 < n <= 128), held in registers all at once: the edges of n and of the
k-steps for every kind of operand, ties, and the sums in 64 bits that decide where half-precision parts cannot."""
import numpy as np
import pytest

from oracle import sweep as osweep
from paper_2605_18856_amd import bsse, workloads
from tests import kernels
from tests.test_gpu_parity import _full_check

pytestmark = pytest.mark.gpu
PATHS = {"normal": "mfma_split6", "int": "mfma_split3", "bf16": "mfma_bf16"}


@pytest.mark.parametrize("kind", ["normal", "int", "bf16"])
@pytest.mark.parametrize("m", [3, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128])
@pytest.mark.parametrize("n", [33, 63, 64, 65, 96, 97, 127, 128])
def test_edges(m, n, kind):
    if m * n <= 64 or (n == 64 and m <= 32 and kind != "bf16"):
        pytest.skip("another kernel's shape")
    storage = "bf16" if kind == "bf16" else "f32"
    game = workloads.small_game(m, n, 3, 400 + m + n, "normal" if kind == "bf16" else kind, storage)
    for count in (1, 33, 2050):
        X = workloads.host_candidates(m, count, 401 + count, "dirichlet")
        rep, _ = _full_check(game, X, bsse.BSSE_PATH_AUTO, PATHS[kind])
        assert rep.br_mismatch == rep.flagged


@pytest.mark.parametrize("kind", ["dyadic", "vertex"])
@pytest.mark.parametrize("shape", [(20, 40, 2), (50, 64, 2), (100, 33, 2), (40, 90, 2), (60, 20, 3)], ids=lambda s: "m%dn%dK%d" % s)
def test_ties_here_and_there(shape, kind):
    """Whole numbers of thirteen bits, dyadic rows: every sum is exact.  Two columns, in different row tiles where there
    are two, are equal and win for rows with most on the first leader action only: the ties are the oracle's."""
    m, n, K = shape
    rng = np.random.default_rng(410 + m)
    game = workloads.small_game(m, n, K, 411, "normal")
    game.A = rng.integers(-4000, 4000, game.A.shape).astype(np.float32)
    game.B = rng.integers(-4000, 4000, game.B.shape).astype(np.float32)
    game.B[:, 0, 3] = 4095.0
    game.B[:, 1:, 3] = -4001.0
    game.B[:, :, n - 1] = game.B[:, :, 3]
    assert kernels.half_parts(game) == (m > 32)
    X = workloads.host_candidates(m, 3001, 412, kind)
    X[::7] = 0.0
    X[::7, 0] = 1.0
    rep, out = _full_check(game, X, bsse.BSSE_PATH_AUTO, "mfma_split6")
    assert rep.br_mismatch == 0
    ref = osweep.sweep(game.A, game.B, game.prior, X, diagnostics=True)
    assert out.n_tie_evals == int((ref.gap == 0).sum()) > 0
