"""The kernels that find a brick's faces from its face flags (divergence,
velocity update, per-face gradient, coefficient assembly) against the oracle,
on octrees whose bricks meet walls, finer and coarser leaves in many
combinations, and whose leaf bricks do not fill a workgroup's groups."""

import warnings

import numpy as np
import pytest

import problems
from gpu_fixtures import Case
from oracle import projection as PJ

pytestmark = pytest.mark.gpu


def _spec(seed):
    """Random spheres and boxes, some at the walls and corners."""
    rng = np.random.default_rng(seed)
    prims = []
    for _ in range(3):
        if rng.random() < 0.5:
            prims.append(problems.sphere_prim(rng.uniform(0, 1, 3), rng.uniform(0.02, 0.3)))
        else:
            lo = rng.uniform(-0.1, 0.8, 3)
            prims.append(problems.box_prim(lo, lo + rng.uniform(0.05, 0.4, 3)))
    lmin = int(rng.integers(2, 4))
    return {"min_level": lmin, "max_level": lmin + int(rng.integers(1, 4)), "node_size": 4,
            "prims": prims}


SPECS = {**{f"random{s}": _spec(s) for s in range(4)},
         "one_brick": problems.uniform_spec(2),
         # coarse leaves in the last group of bricks, next to the first inner one
         "far_corner": {"min_level": 3, "max_level": 4, "node_size": 4,
                        "prims": [problems.sphere_prim((1, 1, 1), 0.01)]},
         "corner": {"min_level": 2, "max_level": 5, "node_size": 4,
                    "prims": [problems.sphere_prim((0, 0, 0), 0.01)]}}


@pytest.mark.parametrize("name", list(SPECS))
@pytest.mark.parametrize("device", [False, True])
def test_face_kernels(name, device):
    from paper_2604_18886_amd import mfmg
    rng = np.random.default_rng(5)
    bc = tuple(int(x) for x in rng.integers(0, 2, 6)[:5]) + (1,)
    probe = Case(1, SPECS[name], bc=bc, theta=0.3, rhs=0)
    nf, n = probe.disc.n_faces, probe.T.n
    # closed faces, closed-off cells and ordinary ones
    beta = rng.uniform(0.1, 1.0, nf) * (rng.random(nf) > 0.2)
    solid = rng.random(n) < 0.05
    other = probe.disc.face_other
    beta[solid[probe.disc.face_owner] | ((other >= 0) & solid[np.maximum(other, 0)])] = 0.0
    case = Case(1, SPECS[name], bc=bc, theta=0.3, beta=beta, rhs=rng.uniform(-1, 1, n))
    if device:
        case.tree = mfmg.build_octree(SPECS[name], device=True)
    print(f"  {name}: {n} leaves, {nf} faces", flush=True)
    co = mfmg.assemble_coeffs(case.tree, case.device(beta), bc, 0.3)
    h = mfmg.build_hierarchy(co, coarsest_level=2)
    c = co.leaf_coeffs().cpu().numpy()[0]
    diag = case.disc.A.diagonal() if name == "one_brick" else None
    if diag is not None:  # (at T-junctions A's diagonal holds ghost terms too)
        act = case.disc.active
        assert np.abs((c - diag)[act]).max() <= 1e-14 * np.abs(diag).max()
    assert np.array_equal(c != 0, case.disc.active)
    b_d = case.device(beta)
    u = rng.uniform(-1, 1, nf)
    p = np.where(case.disc.active, rng.uniform(-1, 1, n), 0.0)
    div = mfmg.divergence(h, b_d, case.device(u)).cpu().numpy()
    ref = PJ.divergence(case.disc, beta, u)
    assert np.abs(div - ref).max() <= 1e-14 * np.abs(ref).max()
    u_d = mfmg.project_velocity(h, b_d, case.device(p), case.device(u)).cpu().numpy()
    ref = PJ.project(case.disc, beta, u, p)
    assert np.abs(u_d - ref).max() <= 1e-13 * np.abs(ref).max()
    assert np.array_equal(u_d[beta == 0], u[beta == 0])
    y = mfmg.apply_operator(h, case.device(p)).cpu().numpy()
    ref = case.disc.A @ p
    assert np.abs(y - ref).max() <= 1e-13 * np.abs(ref).max()
    # the gradient of whatever lambda one iteration gives
    g = np.where(case.disc.active, rng.uniform(-1, 1, n), 0.0)
    with warnings.catch_warnings():
        warnings.simplefilter("ignore", mfmg.NotConvergedWarning)
        lam, grad, _ = mfmg.pcg_solve_adjoint(h, case.device(p), case.device(g), max_iter=1)
    ref = case.disc.face_gradient(lam.cpu().numpy(), p)
    assert np.abs(grad.cpu().numpy() - ref).max() <= 1e-13 * np.abs(ref).max()
