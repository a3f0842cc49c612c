"""The composite operator and its transpose do not depend on the restriction
scale alpha of the hierarchy they are applied through: A and A^T against the
oracle's matrix, and the solutions of both systems."""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case, rel
from oracle import krylov as K

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=["cut_sphere_4_6", "box_5_7"])
def case(request):
    if request.param == "cut_sphere_4_6":
        return Case(5, problems.config_spec(5, 4, 6))
    # (the box meets walls: leaves with an inner neighbour and a plus wall)
    spec = {"min_level": 5, "max_level": 7, "node_size": 4,
            "prims": [problems.box_prim((0.1, 0.55, 0.55), (0.45, 1.0, 0.97))]}
    return Case(3, spec, bc=(1, 0, 0, 1, 1, 0), theta=0.4)


@pytest.mark.parametrize("alpha,beta_mg", [(1.0, 1.0), (3.0, 3.0), (4.0, 2.0)])
@pytest.mark.parametrize("precision", [0, 1])
def test_operator_is_the_same_for_any_alpha(case, precision, alpha, beta_mg):
    from paper_2604_18886_amd import mfmg
    h = case.gpu_hierarchy(precision=precision, alpha=alpha, beta_mg=beta_mg)
    x = np.where(case.disc.active, np.random.default_rng(6).uniform(-1, 1, case.T.n), 0.0)
    for transpose, A in ((False, case.disc.A), (True, case.disc.A.T)):
        y = mfmg.apply_operator(h, case.device(x), transpose=transpose).cpu().numpy()
        want = A @ x
        assert np.abs(y - want).max() <= 1e-13 * np.abs(want).max(), transpose


@pytest.mark.parametrize("precision", [0, 1])
def test_solutions_with_another_alpha(case, precision):
    from paper_2604_18886_amd import mfmg
    h = case.gpu_hierarchy(precision=precision, alpha=1.9, beta_mg=1.9)
    p, st = mfmg.pcg_solve(h, case.device(case.rhs), rtol=1e-11)
    assert st["status"] == mfmg.OK
    x, _ = case.oracle_solve(1e-13)
    assert rel(p.cpu().numpy(), x) <= 1e-8
    lam, _, st = mfmg.pcg_solve_adjoint(h, p, case.device(case.rhs), rtol=1e-11)
    assert st["status"] == mfmg.OK
    y, _ = K.pcg(case.disc.A.T.tocsr(), case.rhs, case.hier.vcycle_T, 1e-13, 400,
                 active=case.disc.active)
    assert rel(lam.cpu().numpy(), y) <= 1e-8
