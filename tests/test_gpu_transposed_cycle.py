"""The transposed cycle in solution form against the oracle's transposed
cycle, over what its branches depend on: cycle index (a level visited once or
several times), smoothing counts, the bottom of the cycle in one kernel or in
separate ones, leaves on the coarsest level and on the one above it, walls."""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case, rel
from oracle import multigrid as M

pytestmark = pytest.mark.gpu

CASES = {
    # leaves on the coarsest level, T-junctions on the level above it
    "cut_sphere_3_5": lambda: Case(3, problems.config_spec(3, 3, 5)),
    # no leaves on the coarsest level, leaves without T-junctions above it
    "cut_sphere_4_6": lambda: Case(3, problems.config_spec(3, 4, 6)),
    # no leaves on the two coarsest levels, all walls Dirichlet
    "sphere_band_5_6": lambda: Case(2, problems.config_spec(2, 5, 6)),
    # two levels, no T-junction
    "uniform16": lambda: Case(1, problems.uniform_spec(4)),
}
PARAMS = [dict(mu=1), dict(mu=2), dict(mu=3, nu_pre=1, nu_post=2, nu_coarse=3),
          dict(mu=2, nu_pre=2, nu_post=0), dict(mu=2, nu_pre=0, nu_post=1)]


@pytest.fixture(scope="module", params=list(CASES))
def case(request):
    print(f"\n[case {request.param}]", flush=True)
    return CASES[request.param]()


# bottom "1"/"0": the bottom of the cycle in one kernel or in separate ones;
# "p": separate, and the prolongation in a pass of its own
@pytest.mark.parametrize("bottom", ["1", "0", "p"])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("prm", PARAMS, ids=[str(i) for i in range(len(PARAMS))])
def test_transposed_cycle(case, prm, precision, bottom):
    from paper_2604_18886_amd import mfmg
    H = M.Hierarchy(case.disc, coarsest=3, **prm)
    env = {"MFMG_FUSE_BOTTOM": "1" if bottom == "1" else "0",
           "MFMG_FUSE_PROLONG": "0" if bottom == "p" else "1"}
    with pytest.MonkeyPatch.context() as mp:
        for k, v in env.items():
            mp.setenv(k, v)
        h = case.gpu_hierarchy(precision=precision, **prm)
    rng = np.random.default_rng(77)
    r = np.where(case.disc.active, rng.uniform(-1, 1, case.T.n), 0.0)
    for _ in range(2):  # the second call finds the first one's arrays
        z = mfmg.apply_precond(h, case.device(r), transpose=True).cpu().numpy()
        want = (H if precision == 0 else H.stored_precision()).vcycle_T(r)
        err = rel(z, want)
        print(f"  {prm} precision={precision} bottom={bottom}: {err:.2e}", flush=True)
        # FP64 rounding; FP32 rounding of a cycle of a few hundred operations
        # per cell
        assert err <= (1e-12 if precision == 0 else 1e-5)
