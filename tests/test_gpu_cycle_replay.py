"""Cycles replayed from a handle's graph: the time amg_vcycle holds its caller's
thread, a caller's own capture, and mixed-precision and split-residual handles
solved side by side against handles that launch every kernel.

Every test prints the case it runs (flushed) before touching the GPU."""
import time

import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU-only machines
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2202_11288_amd import binding as B  # noqa: E402

CONST, DELTA = B.kernel(B.AMG_K_CONST), 0.07


def vector(N, seed, dtype=torch.float64):
    return torch.from_numpy(synthetic.random_vector(2 * N - 1, seed=seed)).to("cuda", dtype)


def test_vcycle_holds_the_caller_less_than_its_launches():
    """A replayed cycle of 60 and more kernels is one graph launch to the caller's
    thread (a fifth of the kernels' launches; half of them is the bound)."""
    N = 2 ** 17
    print("[case] host time", N, flush=True)
    r = vector(N, 1)
    e = torch.empty_like(r)
    took = []
    for flags in (0, B.AMG_FLAG_EAGER):
        h = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(flags=flags, m1=2, m2=2))
        try:
            ts = []
            for k in range(40):
                t0 = time.perf_counter()
                B.amg_vcycle(h, r, e)
                ts.append(time.perf_counter() - t0)
                torch.cuda.synchronize()
            took.append(np.median(ts[10:]))
        finally:
            B.amg_destroy(h)
    print("[case] us", [t * 1e6 for t in took], flush=True)
    assert took[0] < 0.5 * took[1]


@pytest.mark.parametrize("cycle", [1, 2])
@pytest.mark.parametrize("prec,dtype", [(B.AMG_FP64, torch.float64),
                                        (B.AMG_MIXED, torch.float32)])
def test_callers_capture(prec, dtype, cycle):
    """A caller captures a cycle of a handle that replays its own."""
    N = 2 ** 14
    print("[case] capture", prec, cycle, flush=True)
    h = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(precision=prec, cycle=cycle))
    try:
        r = vector(N, 2, dtype)
        want, e = torch.empty_like(r), torch.empty_like(r)
        for _ in range(3):
            B.amg_vcycle(h, r, want)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            B.amg_vcycle(h, r, e)
        for k in range(4):
            e.fill_(float("nan"))
            g.replay()
            assert torch.equal(e, want), k
            other = torch.empty_like(r)
            B.amg_vcycle(h, 2 * r, other)
            assert torch.equal(other, 2 * want), k  # a power of two: exact
        del g
    finally:
        B.amg_destroy(h)


@pytest.mark.parametrize("opts", [dict(inner=B.AMG_INNER_GMRES), dict(cycle=2),
                                  dict(flags=B.AMG_FLAG_ACCURATE_RESIDUAL)],
                         ids=["gmres", "wcycle", "split"])
def test_mixed_handles_side_by_side(opts):
    """The same bits and histories from replayed FP32 cycles, several times, with
    other work in between."""
    N = 2 ** 14
    print("[case] side by side", opts, flush=True)
    o = dict(opts, precision=B.AMG_MIXED)
    bs = [vector(N, k) for k in range(3)]
    hs = [B.amg_setup(CONST, DELTA, N, B.amg_default_opts(**o)) for _ in bs]
    he = B.amg_setup(CONST, DELTA, N, B.amg_default_opts(
        **dict(o, flags=o.get("flags", 0) | B.AMG_FLAG_EAGER)))
    try:
        want = []
        for b in bs:
            x = torch.zeros_like(b)
            B.amg_solve(he, b, x, 1e-9)
            want.append((x, np.array(B.amg_residual_history(he))))
        for _ in range(3):
            xs = [torch.zeros_like(b) for b in bs]
            B.amg_solve_batch(hs, bs, xs, [1e-9] * len(bs))
            for (x, k), y, h in zip(want, xs, hs):
                assert torch.equal(x, y)
                assert np.array_equal(k, np.array(B.amg_residual_history(h)))
            _ = (xs[0] * 2).sum().item()
    finally:
        for h in hs + [he]:
            B.amg_destroy(h)
