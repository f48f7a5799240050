"""Solves that end sooner than most: no V-cycle runs behind the round that ends
them, whether the handle has solved before or not.

Every test prints the case it runs (flushed) before touching the GPU."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU-only machines
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2202_11288_amd import binding as B  # noqa: E402


@pytest.mark.parametrize("inner", [B.AMG_INNER_VCYCLE, B.AMG_INNER_PCG])
def test_time_step_of_one_cycle(inner):
    """A time step from the state before it, whose first cycle ends it, against a
    handle that queues nothing ahead (profiled): the same bits, and no longer.  A
    second cycle would be two fifths more; a sixth is allowed for."""
    N = 2 ** 20
    print("[case] step of one cycle", inner, flush=True)
    kern, tau = B.kernel(B.AMG_K_CONST), 1.0 / N
    x = np.concatenate([np.arange(1, N) / N, (np.arange(N) + 0.5) / N])
    u = x * x * (1 - x) ** 2
    f = B.amg_manufactured_rhs(kern, 0.25, N)
    hist = [torch.from_numpy(np.exp(j * tau) * u).cuda() for j in (3, 2, 1, 0)]
    src = torch.from_numpy(tau * np.exp(4 * tau) * (u + 2.0 * f)).cuda()
    took, first, outs = [], [], []
    for flags in (0, B.AMG_FLAG_PROFILE):
        o = B.amg_default_opts(inner=inner, shift=25.0 / 12.0, scale=2.0 * tau, flags=flags)
        ts = []
        for _ in range(6):  # each handle's first step, and those behind it
            h = B.amg_setup(kern, 0.25, N, o)
            try:
                xo = torch.empty_like(hist[0])
                for _ in range(4):
                    torch.cuda.synchronize()
                    t0 = time.perf_counter()
                    out = B.amg_bdf4_step(h, hist, src, xo, 1e-8)
                    ts.append(time.perf_counter() - t0)
            finally:
                B.amg_destroy(h)
        assert out[:2] == (B.AMG_OK, 1)
        first.append(np.median(ts[4::4]))
        took.append(np.median([t for k, t in enumerate(ts) if k % 4]))
        outs.append((out, xo.clone()))
    print("[case] us, first", [t * 1e6 for t in first], "then", [t * 1e6 for t in took], flush=True)
    assert outs[0][0] == outs[1][0] and torch.equal(outs[0][1], outs[1][1])
    assert first[0] < 7 / 6 * first[1] and took[0] < 7 / 6 * took[1]
