"""Complete levels of 16^3 to 64^3 cells in tiles with a halo, as the finest
level (all leaves), as an inner level without leaves and as one with both,
against the oracle's cycle: every wall condition (the halo is cut at the
walls), inactive cells, one and two smoothing iterations on either side (the
halo holds two; three take the separate kernels), V- and W-cycles, both
directions."""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case, rel
from oracle import multigrid as M

pytestmark = pytest.mark.gpu

BC = {"mixed": (1, 0, 0, 1, 1, 0), "neumann": (0,) * 6}


@pytest.mark.parametrize("walls", list(BC))
@pytest.mark.parametrize("levels", [(4, 4), (5, 5), (6, 6), (5, 6), (6, 7)])
@pytest.mark.parametrize("precision,mu,nu", [(0, 1, (2, 2)), (0, 2, (1, 2)), (1, 1, (2, 1)),
                                             (1, 2, (2, 2)), (1, 1, (1, 1)), (0, 1, (3, 2))])
def test_cycle_with_tiles(levels, walls, precision, mu, nu):
    from paper_2604_18886_amd import mfmg
    spec = {"min_level": levels[0], "max_level": levels[1], "node_size": 4,
            "prims": [problems.box_prim((0.1, -0.1, 0.55), (0.45, 0.3, 0.9))]}
    probe = Case(1, spec, bc=BC[walls], theta=0.4, rhs=0)
    rng = np.random.default_rng(23)
    beta = rng.uniform(0.05, 1.0, probe.disc.n_faces)
    x = (probe.T.ijk + 0.5) * np.ldexp(1.0, -probe.T.level.astype(int))[:, None]
    solid = ((x - 0.3) ** 2).sum(1) < 0.04
    other = probe.disc.face_other
    beta[solid[probe.disc.face_owner] | ((other >= 0) & solid[np.maximum(other, 0)])] = 0.0
    case = Case(1, spec, bc=BC[walls], theta=0.4, beta=beta, rhs=0)
    H = M.Hierarchy(case.disc, coarsest=3, mu=mu, nu_pre=nu[0], nu_post=nu[1])
    if precision:
        H = H.stored_precision()
    co = mfmg.assemble_coeffs(case.tree, case.device(beta), BC[walls], 0.4)
    h = mfmg.build_hierarchy(co, coarsest_level=3, mu=mu, nu_pre=nu[0], nu_post=nu[1],
                             precision=precision)
    r = np.where(case.disc.active, rng.uniform(-1, 1, case.T.n), 0.0)
    z = mfmg.apply_precond(h, case.device(r)).cpu().numpy()
    zt = mfmg.apply_precond(h, case.device(r), transpose=True).cpu().numpy()
    e, et = rel(z, H.vcycle(r)), rel(zt, H.vcycle_T(r))
    print(f"  {levels} {walls} precision={precision} mu={mu} nu={nu}: {e:.1e} {et:.1e}",
          flush=True)
    tol = 1e-12 if precision == 0 else 1e-5
    assert e <= tol and et <= tol
