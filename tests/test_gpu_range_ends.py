"""Ends of the accepted ranges: payoffs near the ends of fp32 (no matrix-core path but the listed ones), rows
near them, local sets too large to be generated together or at all, more programs asked for than profiles exist."""
import numpy as np
import pytest

from paper_2605_18856_amd import bsse, workloads
from tests.test_gpu_parity import _full_check, _make, _run_eval

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(9, 8, 5, "f32"), (20, 30, 3, "f32"), (40, 20, 2, "f32"), (24, 7, 3, "bf16")],
                         ids=lambda s: "m%dn%dK%d%s" % s)
@pytest.mark.parametrize("scale, path", [(2.0 ** -124, "valu"), (2.0 ** -90, "mfma"), (2.0 ** 115, "mfma"), (2.0 ** 124, "valu")])
def test_payoffs_of_any_size(shape, scale, path):
    m, n, K, storage = shape
    game = workloads.small_game(m, n, K, 5 + m, kind="normal", storage=storage)
    game.A = np.where(np.abs(game.A) < 2.0 ** -9, 0.0, game.A * np.float32(scale)).astype(np.float32)
    game.B = np.where(np.abs(game.B) < 2.0 ** -9, 0.0, game.B * np.float32(scale)).astype(np.float32)
    _full_check(game, workloads.host_candidates(m, 3001, 8), bsse.BSSE_PATH_AUTO, path)


@pytest.mark.parametrize("m, n, K, cloud, k", [(16, 12, 3, 4096, 4), (128, 9, 2, 300001, 3), (5, 3, 2, 100, 200)])
def test_refine_spelled_out(m, n, K, cloud, k):
    """One round by bsse_refine and by its steps: sets generated together, and one by one (300001 rows of
    128 exceed half of what is held at once)."""
    game = workloads.small_game(m, n, K, 12)
    seed, radius = 77, 0.25
    with _make(game) as g:
        bsse.bsse_dirichlet(g, 3, 0, 5000)
        x, value, br, evals = bsse.bsse_refine(g, k, 1, cloud_count=cloud, seed=seed, radius=radius)
        kept = bsse.candidates_to_host(g)
        bsse.bsse_dirichlet(g, 3, 0, 5000)
        X = bsse.candidates_to_host(g)
        v, i, b = bsse.bsse_sweep_topk(g, k)
        best, bx, bb = v[0], X[i[0]], b[0]
        centres = X[i]
        for c, centre in enumerate(centres):
            bsse.bsse_dirichlet_around(g, seed + c, 0, cloud, centre, radius)
            v, i, b = bsse.bsse_sweep_topk(g, 1)
            if v[0] > best:
                best, bx, bb = v[0], bsse.candidates_to_host(g)[i[0]], b[0]
        assert (value, evals) == (best, (5000 + len(centres) * cloud) * K)
        assert np.array_equal(x, bx) and np.array_equal(br, bb)
        assert np.array_equal(kept, bsse.candidates_to_host(g))          # the last local set stays


def test_refine_refuses_sets_beyond_a_call():
    game = workloads.small_game(16, 4, 2, 12)
    with _make(game) as g:
        bsse.bsse_dirichlet(g, 3, 0, 100)
        for cloud in ((1 << 31) + 1, 1 << 60, 1 << 62):
            with pytest.raises(bsse.BsseError):
                bsse.bsse_refine(g, 2, 1, cloud_count=cloud)
        assert bsse.bsse_refine(g, 2, 1, cloud_count=64)[3] > 0


@pytest.mark.parametrize("n, K", [(1, 4), (2, 3), (7, 1)])
def test_more_programs_than_profiles(n, K):
    game = workloads.small_game(6, n, K, 3)
    with _make(game) as g:
        bsse.bsse_dirichlet(g, 3, 0, 20000)
        few = bsse.bsse_solve_realised(g, max_profiles=n ** K)
        many = bsse.bsse_solve_realised(g, max_profiles=2 ** 31 - 1)
        assert few[0] == many[0] and few[3:] == many[3:] and many[3] <= n ** K


@pytest.mark.parametrize("shape", [(9, 8, 5), (20, 13, 3), (30, 40, 3), (40, 20, 2), (70, 12, 2), (100, 90, 2), (128, 5, 3)],
                         ids=lambda s: "m%dn%dK%d" % s)
@pytest.mark.parametrize("kind, exponent", [("normal", e) for e in (-124, -112, -100, -61, 99, 101, 126, 128)] +
                         [("int", -126), ("int", 128)])
def test_rows_of_any_size(shape, kind, exponent):
    """Rows at both ends of fp32 on the any-shape kernel, ordinary ones between them: no further from the
    64-bit value than the vector unit's sum of the same numbers.  An fp32 sum of m terms is off by at most
    m 2^-24 of their absolute sum; at the lower end the products themselves are rounded to multiples of
    2^-149, each by half of one at most (once per part product, and once more where a payoff is scaled back)."""
    m, n, K = shape
    game = workloads.small_game(m, n, K, 7 + m, kind=kind)
    small = np.float32(2.0 ** -12 if exponent > 90 else 2.0 ** -4)             # (sums stay below the greatest number)
    game.A, game.B = game.A * small, game.B * small
    X = workloads.host_candidates(m, 700, 8)
    X[::2] *= (np.float64(2.0) ** exponent / X[::2].max(axis=1, keepdims=True)).astype(np.float64) * (1.0 - 2.0 ** -23)
    with _make(game) as g, _make(game, bsse.BSSE_PATH_VALU) as v:
        assert bsse.bsse_path_name(g) == ("mfma_split3" if kind == "int" else "mfma_split6")
        Xd, V, br = _run_eval(g, X)
        _, Vv, brv = _run_eval(v, X)
        out = bsse.bsse_sweep(g, Xd, len(X))
        assert (out.best_index, np.float32(out.best_value)) == (int(np.argmax(V)), V.max())
    A, p, X = game.A.astype(np.float64), game.prior.astype(np.float64), X.astype(np.float64)
    B = game.B.astype(np.float64)

    def off(V, br):
        """Error of the values, and how far the actions are from the best ones, over what is allowed."""
        exact = np.zeros(len(X))
        scale = np.zeros(len(X))
        for t in range(K):
            terms = X * A[t][:, br[:, t]].T
            exact += p[t] * terms.sum(axis=1)
            scale += p[t] * np.abs(terms).sum(axis=1)
            u = X @ B[t]
            gap = u.max(axis=1) - u[np.arange(len(X)), br[:, t]]
            assert np.all(gap <= 2 * (m * 2.0 ** -24 * (np.abs(X) @ np.abs(B[t])).max(axis=1) + 6 * m * 2.0 ** -150))
        return np.abs(V - exact) / ((m + K) * 2.0 ** -24 * scale + (6 * m + K + 1) * 2.0 ** -150)

    assert off(V, br).max() <= 1.0 and off(Vv, brv).max() <= 1.0
