"""The bottom of the cycle in one kernel on the grids it can meet: levels 4
and 3 (16^3 and 8^3 cells) or 3 and 2, with every wall condition, inactive
cells and leaves on the finer of the two, against the oracle's cycle."""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case, rel
from oracle import multigrid as M

pytestmark = pytest.mark.gpu

BC = {"mixed": (1, 0, 0, 1, 1, 0), "neumann": (0,) * 6, "dirichlet": (1,) * 6}


@pytest.mark.parametrize("walls", list(BC))
@pytest.mark.parametrize("lc,levels", [(3, (4, 5)), (2, (3, 4)), (2, (4, 5)), (3, (5, 6))])
@pytest.mark.parametrize("precision,mu", [(0, 1), (1, 1), (1, 2), (0, 2)])
def test_cycle_with_one_kernel_bottom(lc, levels, walls, precision, mu):
    from paper_2604_18886_amd import mfmg
    spec = {"min_level": levels[0], "max_level": levels[1], "node_size": 4,
            "prims": [problems.box_prim((0.1, -0.1, 0.55), (0.45, 0.3, 0.9))]}
    probe = Case(1, spec, bc=BC[walls], theta=0.4, rhs=0)
    rng = np.random.default_rng(17)
    beta = rng.uniform(0.05, 1.0, probe.disc.n_faces)
    x = (probe.T.ijk + 0.5) * np.ldexp(1.0, -probe.T.level.astype(int))[:, None]
    solid = ((x - 0.3) ** 2).sum(1) < 0.04
    other = probe.disc.face_other
    beta[solid[probe.disc.face_owner] | ((other >= 0) & solid[np.maximum(other, 0)])] = 0.0
    case = Case(1, spec, bc=BC[walls], theta=0.4, beta=beta, rhs=0)
    H = M.Hierarchy(case.disc, coarsest=lc, mu=mu)
    if precision:
        H = H.stored_precision()
    co = mfmg.assemble_coeffs(case.tree, case.device(beta), BC[walls], 0.4)
    h = mfmg.build_hierarchy(co, coarsest_level=lc, mu=mu, precision=precision)
    r = np.where(case.disc.active, rng.uniform(-1, 1, case.T.n), 0.0)
    z = mfmg.apply_precond(h, case.device(r)).cpu().numpy()
    zt = mfmg.apply_precond(h, case.device(r), transpose=True).cpu().numpy()
    e, et = rel(z, H.vcycle(r)), rel(zt, H.vcycle_T(r))
    print(f"  lc={lc} {levels} {walls} precision={precision} mu={mu}: {e:.1e} {et:.1e}",
          flush=True)
    tol = 1e-12 if precision == 0 else 1e-5
    assert e <= tol and et <= tol
