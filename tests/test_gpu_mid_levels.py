"""The mid-size levels' passes (8 elements to a thread) at every geometry the
tuner can choose, symmetric and general spectra, both precisions, with the
volume's edges in play: products, smoothing, residuals and transfers.

Every test prints the case it runs (flushed) before touching the GPU."""
import sys

import numpy as np
import pytest

import synthetic
from oracle import discretize as D
from oracle import tpx
from oracle.dense import Options

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU-only machines
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2202_11288_amd import binding as B  # noqa: E402

CASES = {"const": (B.kernel(B.AMG_K_CONST), D.Kernel(D.CONST, 0.07)),
         "weighted": (B.kernel(B.AMG_K_WEIGHTED, wl=1.2, wr=0.8),
                      D.Kernel(D.WEIGHTED, 0.07, wl=1.2, wr=0.8))}
EPS, EPS32 = np.finfo(np.float64).eps, np.finfo(np.float32).eps


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


# (log2 L, log2 of the row length, columns to a tile): each row length 128..1024
# with each column length 64..512, where a plan pairs them
GEOMETRIES = [(13, 7, 4), (14, 7, 4), (14, 8, 4), (15, 8, 4), (16, 8, 4), (16, 9, 4), (17, 8, 4),
              (17, 9, 4), (18, 9, 4), (18, 10, 4), (19, 10, 4)]


@pytest.mark.parametrize("geom", GEOMETRIES, ids=lambda g: "L%d-%d-%d" % g)
@pytest.mark.parametrize("name", list(CASES))
def test_products_and_cycles(name, geom):
    """An FFT product's relative error in the 2-norm stays within
    2 eps (2 + log2 L); a V-cycle's within that of its products, 8 to a level
    at two sweeps a side (the conditioning of these kernels' coarsest level,
    about 10, included)."""
    logL, logL1, tcols = geom
    print("[case] mid", name, geom, flush=True)
    sys.stdout.flush()
    kern, okern = CASES[name]
    N = 2 ** (logL - 1)
    H = tpx.Hierarchy.build(tpx.from_stencil(okern, N), 5)
    x = synthetic.random_vector(2 * N - 1, seed=logL).astype(np.float32).astype(np.float64)
    yr = H.levels[0].matvec(x)
    er = tpx.vcycle(H, x, Options(m1=2, m2=2))
    bound = 2 * (2 + logL)
    B.amg_plan_set(logL, logL1, tcols)
    try:
        for prec, dtype, eps in ((B.AMG_FP64, torch.float64, EPS),
                                 (B.AMG_MIXED, torch.float32, EPS32)):
            h = B.amg_setup(kern, 0.07, N, B.amg_default_opts(precision=prec, m1=2, m2=2))
            try:
                xd = torch.from_numpy(x).to("cuda", dtype)
                y = torch.full_like(xd, float("nan"))
                (B.amg_level_matvec if eps == EPS else B.amg_level_matvec_f32)(h, 0, xd, y)
                err = np.linalg.norm(host(y) - yr) / np.linalg.norm(yr)
                assert err < bound * eps, (prec, err)
                e = torch.full_like(xd, float("nan"))
                for _ in range(3):  # direct launches, then the captured cycle
                    B.amg_vcycle(h, xd, e)
                    err = np.linalg.norm(host(e) - er) / np.linalg.norm(er)
                    assert err < 8 * 10 * bound * eps, (prec, err)
                if eps == EPS:
                    r = torch.full_like(xd, float("nan"))
                    b = torch.ones_like(xd)
                    B.amg_residual(h, b, xd, r)
                    rr = 1.0 - yr
                    assert np.linalg.norm(host(r) - rr) < 2 * bound * eps * np.linalg.norm(rr)
            finally:
                B.amg_destroy(h)
    finally:
        B.amg_plan_set(logL)
