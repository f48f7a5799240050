"""The small-level kernel's steps on levels with a band (weakly singular model)
beside those without: what the band's product may add to them.

Every test prints the case it runs (flushed) before touching the GPU."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU-only machines
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2202_11288_amd import binding as B  # noqa: E402


def test_band_steps_take_little_more():
    """A W-cycle handle's set-up is 511 runs of the small levels' step program; with
    a band each step makes one more round trip to memory.  1.57 times the time of
    the same program without a band is what the loads one by one took."""
    N = 2 ** 9
    opts = B.amg_default_opts(cycle=2)
    took = []
    for kern in (B.kernel(B.AMG_K_WEAKLY_SINGULAR, gamma=0.5), B.kernel(B.AMG_K_CONST)):
        print("[case] W set-up", kern.kind, flush=True)
        ts = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            h = B.amg_setup(kern, 0.1, N, opts)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t0)
            B.amg_destroy(h)
        took.append(np.median(ts[1:]))
    print("[case] ms", [t * 1e3 for t in took], took[0] / took[1], flush=True)
    assert took[0] < 1.45 * took[1]
