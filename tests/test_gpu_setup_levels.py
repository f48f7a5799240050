"""Hierarchies formed on the device, level by level against the oracle: sizes
whose coarsening is one workgroup's from the start, from a coarse level on and
at the line between, spectra of small and four-step levels, FP32 copies, and
work arrays that start cleared.

Every test prints the case it runs (flushed) before touching the GPU."""
import numpy as np
import pytest

import synthetic
from oracle import discretize as D
from oracle import tpx

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU-only machines
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2202_11288_amd import binding as B  # noqa: E402

CASES = {"const": (B.kernel(B.AMG_K_CONST), D.Kernel(D.CONST, 0.07)),
         "weighted": (B.kernel(B.AMG_K_WEIGHTED, wl=1.2, wr=0.8),
                      D.Kernel(D.WEIGHTED, 0.07, wl=1.2, wr=0.8))}
EPS, EPS32 = np.finfo(np.float64).eps, np.finfo(np.float32).eps


@pytest.mark.parametrize("logN", [6, 10, 12, 13, 15])
@pytest.mark.parametrize("name", list(CASES))
def test_every_level_matches_the_oracle(name, logN):
    """A level's FFT product stays within 2 eps (2 + log2 L) of the oracle's in
    the 2-norm; Lemma 3.1 adds 8 roundings of an entry per level to either
    side's hierarchy."""
    print("[case] levels", name, logN, flush=True)
    kern, okern = CASES[name]
    N = 2 ** logN
    H = tpx.Hierarchy.build(tpx.from_stencil(okern, N), 5)
    for prec, dtype, eps in ((B.AMG_FP64, torch.float64, EPS),
                             (B.AMG_MIXED, torch.float32, EPS32)):
        h = B.amg_setup(kern, okern.delta, N, B.amg_default_opts(precision=prec))
        try:
            assert B.amg_num_levels(h) == len(H.levels)
            for l, lev in enumerate(H.levels):
                m = B.amg_level_size(h, l)
                x = synthetic.random_vector(m, seed=l + 1).astype(np.float32).astype(np.float64)
                xd = torch.from_numpy(x).to("cuda", dtype)
                y = torch.empty_like(xd)
                mv = B.amg_level_matvec if prec == B.AMG_FP64 else B.amg_level_matvec_f32
                mv(h, l, xd, y)
                want = lev.matvec(x) if l < len(H.levels) - 1 else lev.dense() @ x
                bound = 2 * (2 + (logN + 1 - l)) * eps + 16 * l * EPS
                got = y.cpu().numpy().astype(np.float64)
                assert np.linalg.norm(got - want) <= bound * np.linalg.norm(want), (prec, l)
            # a first cycle of zero on arrays nothing has written: exactly zero
            z = torch.zeros(2 * N - 1, device="cuda", dtype=dtype)
            e = torch.full_like(z, 3.0)
            B.amg_vcycle(h, z, e)
            assert torch.count_nonzero(e).item() == 0
        finally:
            B.amg_destroy(h)
