"""Cross vectors in the large column tiles, which read them only within the bound
that a level's horizon sets to their support: the column and the row they form
against the oracle's, on the two finest levels, with the tiles of the largest
levels chosen for sizes whose oracle is cheap.

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

LOGN = 18
N = 2 ** LOGN
CASES = {"const": (B.kernel(B.AMG_K_CONST), D.CONST, {}),
         "weighted": (B.kernel(B.AMG_K_WEIGHTED, wl=1.2, wr=0.8), D.WEIGHTED,
                      dict(wl=1.2, wr=0.8))}
EPS, EPS32 = np.finfo(np.float64).eps, np.finfo(np.float32).eps
# the horizon in grid steps: one, a few, an odd size, and on either side of
# half the interval, from where on the bound says nothing (level 1: a few steps earlier)
STEPS = [1.0, 3.7, 0.0123 * N, N / 2 - 10.0, N / 2 - 4.0, N / 2 - 1.0]


def check(C, y, row, u, tol_col, tol_row, what):
    """y: the product with the unit vector at w_o; row: (y_o, its input u)."""
    col = np.concatenate([C.p, [C.o], C.xi])
    assert np.abs(y - col).max() <= tol_col * np.abs(col).max(), what
    r = np.concatenate([C.q, [C.o], C.zeta])
    assert abs(row - r @ u) <= tol_row * np.abs(r * u).sum(), what


def edges_seen(C, tol):
    """Whether the outermost entries of the support, which a bound too small by
    one entry would drop, are far above the column's tolerance."""
    col = np.concatenate([C.p, [C.o], C.xi])
    for v in (C.p, C.xi):
        nz = np.flatnonzero(v)
        for part in (nz[nz < C.n // 2], nz[nz >= C.n // 2][::-1]):
            if len(part) and np.abs(v[part[-2:]]).max() <= 4 * tol * np.abs(col).max():
                return False
    return True


@pytest.mark.parametrize("tiles", [[(19, 9, 8), (18, 9, 8)], [(19, 8, 4), (18, 9, 8)]],
                         ids=["columns1024x8", "columns2048x4"])
@pytest.mark.parametrize("name", list(CASES))
def test_column_and_row_within_the_support(name, tiles):
    kern, kind, par = CASES[name]
    try:
        for t in tiles:
            B.amg_plan_set(*t)
        for steps in STEPS:
            print("[case] support", name, tiles, steps, flush=True)
            okern = D.Kernel(kind, steps / N, **par)
            levels = [tpx.from_stencil(okern, N)]
            levels.append(tpx.coarsen(levels[0]))
            for prec, dtype, eps in ((B.AMG_FP64, torch.float64, EPS),
                                     (B.AMG_MIXED, torch.float32, EPS32)):
                h = B.amg_setup(kern, steps / N, N, B.amg_default_opts(precision=prec))
                mv = B.amg_level_matvec if prec == B.AMG_FP64 else B.amg_level_matvec_f32
                try:
                    for l, C in enumerate(levels):
                        m = B.amg_level_size(h, l)
                        tol = eps + 16 * (l + 1) * EPS  # an entry's roundings
                        assert edges_seen(C, tol), (steps, prec, l)
                        x = torch.zeros(m, device="cuda", dtype=dtype)
                        x[C.n] = 1.0
                        y = torch.empty_like(x)
                        mv(h, l, x, y)
                        col = y.cpu().numpy().astype(np.float64)
                        u = synthetic.random_vector(m, seed=l + 7).astype(np.float32)
                        mv(h, l, torch.from_numpy(u).to("cuda", dtype), y)
                        # the row: a sum of m products, each rounded, in tree order
                        check(C, col, y[C.n].item(), u.astype(np.float64), tol,
                              (2 + LOGN) * eps + 16 * (l + 1) * EPS, (steps, prec, l))
                finally:
                    B.amg_destroy(h)
    finally:
        for t in tiles:
            B.amg_plan_set(t[0])
