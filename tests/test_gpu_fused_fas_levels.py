"""The FAS right-hand side in the first half-sweep of a level (k_smooth_fas)
on the levels that take it: incomplete ones (no tile takes them) below the
finest, with leaves and inner bricks.  Against the oracle's cycle, V- and
W-cycles (whose later visits form it separately), one and three smoothing
iterations."""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case, rel
from oracle import multigrid as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=["cut_sphere_5_8", "sphere_band_4_7"])
def case(request):
    if request.param == "cut_sphere_5_8":
        return Case(3, problems.config_spec(3, 5, 8))
    return Case(2, problems.config_spec(2, 4, 7))


@pytest.mark.parametrize("precision,mu,nu", [(0, 1, (1, 2)), (0, 2, (2, 2)), (1, 1, (3, 1)),
                                             (1, 2, (1, 1))])
def test_levels_with_leaves_match_oracle(case, precision, mu, nu):
    from paper_2604_18886_amd import mfmg
    h = case.gpu_hierarchy(precision=precision, mu=mu, nu_pre=nu[0], nu_post=nu[1])
    taken = []
    for level in range(5, case.T.lmax):
        coords, leaf = h.level_bricks(level)
        if leaf.any() and not leaf.all() and len(coords) < 1 << (3 * (level - 2)):
            taken.append(level)
    assert taken
    H = M.Hierarchy(case.disc, coarsest=3, mu=mu, nu_pre=nu[0], nu_post=nu[1])
    if precision:
        H = H.stored_precision()
    rng = np.random.default_rng(59)
    r = np.where(case.disc.active, rng.uniform(-1, 1, case.T.n), 0.0)
    z = mfmg.apply_precond(h, case.device(r)).cpu().numpy()
    e = rel(z, H.vcycle(r))
    print(f"  levels {taken} precision={precision} mu={mu} nu={nu}: {e:.1e}", flush=True)
    assert e <= (1e-12 if precision == 0 else 1e-5)
