"""M^T is the transpose of M for every restriction scale alpha: x . M y =
y . M^T x on the device.  With alpha other than 2 an inner cell's face
coefficient is not the sum over 2 that the assembled diagonal of a leaf next to
it holds, so the transposed cycle has to divide by the sum of the six face
coefficients there, as the forward half-sweeps do.  (The oracle divides by the
stored diagonal, so it is no reference for such an alpha.)"""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=["cut_sphere_4_6", "box_5_7"])
def case(request):
    if request.param == "cut_sphere_4_6":
        return Case(5, problems.config_spec(5, 4, 6))
    spec = {"min_level": 5, "max_level": 7, "node_size": 4,
            "prims": [problems.box_prim((0.1, -0.1, 0.55), (0.45, 0.3, 0.9))]}
    return Case(1, spec, bc=(1, 0, 0, 1, 1, 0), theta=0.4, rhs=0)


@pytest.mark.parametrize("mu", [1, 2])
@pytest.mark.parametrize("alpha,beta_mg", [(1.0, 1.0), (4.0, 2.0)])
@pytest.mark.parametrize("precision", [0, 1])
def test_transposed_cycle_for_any_alpha(case, precision, alpha, beta_mg, mu):
    from paper_2604_18886_amd import mfmg
    h = case.gpu_hierarchy(precision=precision, alpha=alpha, beta_mg=beta_mg, mu=mu)
    rng = np.random.default_rng(8)
    x, y = (np.where(case.disc.active, rng.uniform(0, 1, case.T.n), 0.0) for _ in range(2))
    My = mfmg.apply_precond(h, case.device(y)).cpu().numpy()
    MTx = mfmg.apply_precond(h, case.device(x), transpose=True).cpu().numpy()
    gap = abs(x @ My - y @ MTx) / (abs(x @ My) + abs(y @ MTx))
    print(f"  precision={precision} alpha={alpha} mu={mu}: {gap:.1e}", flush=True)
    assert gap <= (1e-12 if precision == 0 else 1e-5)
