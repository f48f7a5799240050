"""The one-workgroup kernels of the small levels (L <= 2^12) at the edges of
their geometries, against the oracle: one wavefront to a signal up to L = 512,
alternating LDS buffers at 1024 and 2048, one buffer at 4096; every size of the
dense matrix at the bottom; sweeps that smooth, restrict and prolong.

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

CASES = {"const": (B.kernel(B.AMG_K_CONST), D.Kernel(D.CONST, 0.23)),
         "weighted": (B.kernel(B.AMG_K_WEIGHTED, wl=1.2, wr=0.8),
                      D.Kernel(D.WEIGHTED, 0.23, wl=1.2, wr=0.8))}
EPS, EPS32 = np.finfo(np.float64).eps, np.finfo(np.float32).eps


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def dev(x, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(x)).to(device="cuda", dtype=dtype)


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("name", list(CASES))
def test_products_of_every_small_size(name):
    """L = 2^12 down to 2^3: FP64 and FP32 products and the FP64 residual.
    An FFT product's relative error in the 2-norm is a small multiple of
    eps log2 L: bounded by 2 eps (2 + log2 L) here, twice that for the
    residual of two terms."""
    say("small products", name)
    kern, okern = CASES[name]
    N = 2 ** 11
    Ts = [tpx.from_stencil(okern, N)]
    h = B.amg_setup(kern, 0.23, N, B.amg_default_opts(precision=B.AMG_MIXED, coarsest_log2=2))
    try:
        for l in range(B.amg_num_levels(h)):
            m = B.amg_level_size(h, l)
            A = Ts[-1].dense()
            lg = np.log2(m + 1)
            for dtype, eps, f in ((torch.float64, EPS, B.amg_level_matvec),
                                  (torch.float32, EPS32, B.amg_level_matvec_f32)):
                x = dev(synthetic.random_vector(m, seed=l), dtype)
                y = torch.full_like(x, float("nan"))
                f(h, l, x, y)
                yr = A @ host(x)
                err = np.linalg.norm(host(y) - yr) / np.linalg.norm(yr)
                say("L", m + 1, dtype, "err", err)
                assert err < 2 * eps * (2 + lg), (m, dtype, err)
            if l + 1 < B.amg_num_levels(h):
                Ts.append(tpx.coarsen(Ts[-1]))
    finally:
        B.amg_destroy(h)
    for K in range(3, 12):
        N = 2 ** K
        A = tpx.from_stencil(okern, N).dense()
        h = B.amg_setup(kern, 0.23, N, B.amg_default_opts(coarsest_log2=2))
        try:
            x, b = (synthetic.random_vector(2 * N - 1, seed=K + s) for s in (0, 50))
            r = torch.empty(2 * N - 1, device="cuda", dtype=torch.float64)
            B.amg_residual(h, dev(b), dev(x), r)
            rr = b - A @ x
            assert np.linalg.norm(host(r) - rr) < 4 * EPS * (3 + K) * np.linalg.norm(rr), K
        finally:
            B.amg_destroy(h)


@pytest.mark.parametrize("K,coarsest", [(K, 2) for K in range(3, 13)] +
                         [(9, c) for c in range(3, 8)])
def test_cycles_of_every_small_size(K, coarsest):
    """V- and W-cycles whose finest level is each small size, over every size
    of the dense matrix at the bottom.  Two equally valid hierarchies differ
    by rounding that the coarsest solve amplifies: 64 eps kappa (FP64); in
    FP32 the cycle's own arithmetic, eps_32 (2 + log2 L) per product of the
    4 a level makes, each level's correction entering once."""
    N = 2 ** K
    for name, (kern, okern) in CASES.items():
        H = tpx.Hierarchy.build(tpx.from_stencil(okern, N), coarsest)
        kap = np.linalg.cond(H.levels[-1].dense())
        r = synthetic.random_vector(2 * N - 1, seed=K)
        for cycle, m1, m2 in ((1, 1, 1), (1, 2, 3), (2, 1, 1)):
            ref = tpx.vcycle(H, r.astype(np.float32).astype(np.float64),
                             Options(m1=m1, m2=m2, cycle=cycle))
            for prec, dtype in ((B.AMG_FP64, torch.float64), (B.AMG_MIXED, torch.float32)):
                h = B.amg_setup(kern, 0.23, N, B.amg_default_opts(
                    precision=prec, coarsest_log2=coarsest, m1=m1, m2=m2, cycle=cycle))
                try:
                    e = torch.full((2 * N - 1,), float("nan"), device="cuda", dtype=dtype)
                    B.amg_vcycle(h, dev(r.astype(np.float32), dtype), e)
                    err = np.linalg.norm(host(e) - ref) / np.linalg.norm(ref)
                finally:
                    B.amg_destroy(h)
                tol = (max(1e-13, 64 * EPS * kap) if prec == B.AMG_FP64
                       else 4 * (K - coarsest + 1) * EPS32 * (3 + K) + 4 * EPS32 * kap)
                say(name, "K", K, "coarsest", coarsest, (cycle, m1, m2), dtype, err, tol)
                assert err < tol, (name, K, coarsest, cycle, m1, m2, dtype, err, tol)
