"""Solves whose next V-cycle is queued behind the running round, and whose state
and history the kernels publish, against handles that form every round after
the last one's stop test (profiled handles): the same bits.

Every test prints the case it runs (flushed) before touching the GPU."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU-only machines
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2202_11288_amd import binding as B  # noqa: E402

CONST, DELTA = B.kernel(B.AMG_K_CONST), 0.07
ANY = (B.AMG_OK, B.AMG_NOT_CONVERGED, B.AMG_DIVERGED)


def solve(h, b, tol):
    x = torch.zeros_like(b)
    out = B.amg_solve(h, b, x, tol, allow=ANY)
    return out, x, np.array(B.amg_residual_history(h))


@pytest.mark.parametrize("inner", [B.AMG_INNER_VCYCLE, B.AMG_INNER_PCG, B.AMG_INNER_GMRES])
@pytest.mark.parametrize("prec,N", [(B.AMG_FP64, 2 ** 9), (B.AMG_MIXED, 2 ** 13)])
def test_queued_rounds_equal_rounds_in_turn(inner, prec, N):
    """One handle solves again and again: tolerances whose last round is foretold
    and not, a start that is done at once, an iteration limit in the way and a
    restart length inside the solve."""
    print("[case] queued", inner, prec, N, flush=True)
    b = torch.from_numpy(synthetic.random_vector(2 * N - 1, seed=N)).cuda()
    for opts in (dict(), dict(max_iter=2), dict(max_iter=0), dict(restart=3), dict(cycle=2)):
        o = dict(inner=inner, precision=prec, **opts)
        hq = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(**o))
        hp = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(flags=B.AMG_FLAG_PROFILE, **o))
        try:
            for rhs, tol in ((b, 1e-10), (b, 0.5), (torch.zeros_like(b), 1e-10), (b, 1e-4),
                             (b, 3e-8), (2 * b, 1e-10)):
                q, xq, kq = solve(hq, rhs, tol)
                p, xp, kp = solve(hp, rhs, tol)
                assert q == p, (opts, tol)
                assert torch.equal(xq, xp), (opts, tol)
                assert np.array_equal(kq, kp), (opts, tol)
        finally:
            B.amg_destroy(hq)
            B.amg_destroy(hp)


def test_replayed_cycles_equal_launched_ones():
    """Handles that replay their cycle from a graph: GMRES solves side by side
    (V-cycles) and W-cycles, several times, with other work in between."""
    N = 2 ** 14
    print("[case] replayed", N, flush=True)
    bs = [torch.from_numpy(synthetic.random_vector(2 * N - 1, seed=k)).cuda() for k in range(3)]
    for o in (dict(inner=B.AMG_INNER_GMRES), dict(cycle=2)):
        hs = [B.amg_setup(CONST, DELTA, N, B.amg_default_opts(**o)) for _ in bs]
        he = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(flags=B.AMG_FLAG_EAGER, **o))
        try:
            want = [solve(he, b, 1e-9) for b in bs]
            for _ in range(3):
                xs = [torch.zeros_like(b) for b in bs]
                B.amg_solve_batch(hs, bs, xs, [1e-9] * len(bs))
                for (_, x, k), y, h in zip(want, xs, hs):
                    assert torch.equal(x, y)
                    assert np.array_equal(k, np.array(B.amg_residual_history(h)))
                _ = (xs[0] * 2).sum().item()
        finally:
            for h in hs + [he]:
                B.amg_destroy(h)


def test_history_longer_than_the_published_block():
    """A solve of more rounds than the block behind the state holds."""
    N = 2 ** 7
    print("[case] long history", N, flush=True)
    b = torch.from_numpy(synthetic.random_vector(2 * N - 1, seed=1)).cuda()
    o = dict(max_iter=700, omega_pre=0.02, omega_post=0.02, m1=1, m2=1)
    hq = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(**o))
    hp = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(flags=B.AMG_FLAG_PROFILE, **o))
    try:
        (q, xq, kq), (p, xp, kp) = solve(hq, b, 1e-300), solve(hp, b, 1e-300)
        print("[case] iterations", q, flush=True)
        assert q == p and q[1] > 500
        assert torch.equal(xq, xp) and np.array_equal(kq, kp)
    finally:
        B.amg_destroy(hq)
        B.amg_destroy(hp)
