"""What the margins of the left-out products rest on: a bf16 matrix instruction adds its seventeen terms with
errors of at most 2^-26 of the greatest for each and one rounding.  On a game that is one instruction per
follower payoff (m = 16, bf16 storage) best responses show it: no action wins over one that is ahead by more
than both errors, whatever the order and the sizes of the terms."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _make, _run_eval

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", ["first", "last", "mixed"])
@pytest.mark.parametrize("cancel", [False, True], ids=["sum", "cancelling"])
def test_error_of_one_instruction(slots, cancel):
    m, n, K, count = 16, 32, 200, 1500
    rng = np.random.default_rng(17 + len(slots) + cancel)
    small = {"first": np.arange(m) < 8, "last": np.arange(m) >= 8, "mixed": np.arange(m) % 2 == 1}[slots]
    # pairs of columns that are equal but in the small slots: differences from 2^-27 of the greatest term on
    B = rng.uniform(0.5, 1.0, (K, m, n)) * rng.choice([-1.0, 1.0], (K, m, n))
    B[:, :, 1::2] = B[:, :, 0::2]
    scale = np.ldexp(1.0, -rng.integers(17, 27, (K, 1, n // 2)))
    B[:, small, :] = rng.uniform(-1.0, 1.0, (K, int(small.sum()), n)) * np.repeat(scale, 2, axis=2)
    X = rng.uniform(0.5, 1.0, (count, m))
    if cancel:                                           # a great term and its negative: what is left is small
        B[:, np.flatnonzero(~small)[1], :] = -B[:, np.flatnonzero(~small)[0], :]
        X[:, np.flatnonzero(~small)[1]] = X[:, np.flatnonzero(~small)[0]]
    game = workloads.small_game(m, n, K, 18, "normal", "bf16")
    game.B = workloads.round_to_bf16(B.astype(np.float32))
    X = workloads.round_to_bf16(X.astype(np.float32))
    with _make(game) as g:
        assert bsse.bsse_path_name(g) == "mfma_bf16"
        _, _, br = _run_eval(g, X)
    ahead = close = dropped = 0
    for t in range(K):
        terms = X[:, :, None].astype(np.float64) * game.B[t][None].astype(np.float64)
        S = terms.sum(axis=1)                            # (exact: 16-bit products within 2^30 of each other)
        E = 17 * 2.0 ** -26 * np.abs(terms).max(axis=1) + 2.0 ** -24 * np.abs(S)
        rows, j = np.arange(count), br[:, t]
        assert np.all(S[rows, j] + E[rows, j] >= (S - E).max(axis=1))
        other = j ^ 1
        gap, room = S[rows, j] - S[rows, other], E[rows, j] + E[rows, other]
        ahead += int(((gap > room) & (gap < 8 * room)).sum())
        close += int((np.abs(gap) <= room).sum())
        dropped += int((gap < 0).sum())
    # gaps on either side of the bound, and instructions that did lose something
    assert ahead > K * count // 50 and close > K * count // 50 and dropped > 0
