"""The plans of L = 2^13 .. 2^19 that the mid-size levels' test leaves out: mid-size
columns under rows of 1024 points and more, large tiles, and short rows of either
beside them; with both lists, every plan of those sizes is held against the oracle.

Every test prints the case it runs (flushed) before touching the GPU."""
import pytest

import test_gpu_mid_levels as mid

pytestmark = pytest.mark.gpu

B = mid.B

# (log2 L, log2 of the row length, columns to a tile)
OTHERS = [(15, 9, 4), (16, 10, 4), (17, 10, 4), (17, 11, 4), (18, 9, 8), (18, 11, 4), (18, 12, 4),
          (19, 8, 4), (19, 9, 8), (19, 10, 8), (19, 11, 4), (19, 12, 4)]


def test_both_lists_hold_every_plan():
    print("[case] plans", flush=True)
    plans = []
    for logL in range(13, 20):
        for logL1 in range(1, logL):
            for tcols in (1, 2, 4, 8, 16, 32):
                try:
                    B.amg_plan_set(logL, logL1, tcols)
                    plans.append((logL, logL1, tcols))
                except B.AmgError:
                    pass
        B.amg_plan_set(logL)
    assert sorted(plans) == sorted(mid.GEOMETRIES + OTHERS)


@pytest.mark.parametrize("geom", OTHERS, ids=lambda g: "L%d-%d-%d" % g)
@pytest.mark.parametrize("name", list(mid.CASES))
def test_products_and_cycles_of_the_others(name, geom):
    mid.test_products_and_cycles(name, geom)
