"""Small solves: the kernels that use (r, z) and (p, A p) add the workgroups'
partials themselves (up to 1024 of them, 4096 bricks); above that a launch of
its own does.  On both sides of the line: the oracle's iterates, and the end of
a solve whose (r, z) underflows to 0 before its first step."""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case, rel

pytestmark = pytest.mark.gpu

LEVELS = [(3, 3), (4, 4), (4, 6), (6, 6), (5, 7)]  # 8 to 12503 bricks


def _case(levels, scale=1.0):
    prims = [problems.sphere_prim((0.5, 0.5, 0.5), 0.3, 0.0)] if levels[0] != levels[1] else []
    spec = {"min_level": levels[0], "max_level": levels[1], "node_size": 4, "prims": prims}
    case = Case(1, spec, bc=(1, 0, 0, 1, 1, 0))
    case.beta = case.beta * scale
    return case


@pytest.mark.parametrize("levels", LEVELS)
@pytest.mark.parametrize("precision", [0, 1])
def test_iterates(levels, precision):
    """FP64: as many iterations as the oracle's; both cycles: its solution (the
    FP32 cycle may take more iterations, 12 for 10 at 64^3)."""
    from paper_2604_18886_amd import mfmg
    case = _case(levels)
    x, info = case.oracle_solve(1e-10)
    p = case.device(np.zeros(case.T.n))
    _, st = mfmg.pcg_solve(case.gpu_hierarchy(precision), case.device(case.rhs), p, rtol=1e-10)
    print(f"  {levels} precision={precision}: {st['iters']} iterations", flush=True)
    assert st["status"] == 0
    if precision == 0:
        assert st["iters"] == info["iters"]
    assert rel(p.cpu().numpy(), x) <= 1e-8


@pytest.mark.parametrize("levels", LEVELS)
def test_underflowing_product_stops(levels):
    from paper_2604_18886_amd import mfmg
    case = _case(levels, 1e10)
    rhs = np.zeros(case.T.n)
    rhs[case.T.n // 2] = 1e-160  # ||rhs||^2 = 1e-320; (r, M r) is 1e-10 of it: 0
    p = case.device(np.zeros(case.T.n))
    with pytest.raises(mfmg.MFMGError) as e:
        mfmg.pcg_solve(case.gpu_hierarchy(0), case.device(rhs), p, rtol=1e-10)
    assert e.value.status == -5
