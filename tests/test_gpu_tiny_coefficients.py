"""FP64 coefficients below the normal range.  The cycle's one-kernel levels
(k_bottom, k_tile) divide by a reciprocal, which overflows for a subnormal
diagonal, so such a hierarchy runs the separate kernels.

beta = 2^-1030 and a right-hand side scaled by 2^-400 are powers of two, all
coefficients of the cases are multiples of 2^-1040 with few significant bits,
and no other number leaves the normal range: every result is that of the
unscaled problem times 2^630 for a solution (2^-400 / 2^-1030), bit for bit
against the separate kernels."""

import numpy as np
import pytest

import problems
from gpu_fixtures import Case

pytestmark = pytest.mark.gpu

SPECS = {"uniform32": problems.config_spec(1), "sphere_band_4_6": problems.config_spec(2, 4, 6)}


@pytest.mark.parametrize("name", list(SPECS))
def test_subnormal_diagonals(name, monkeypatch):
    from paper_2604_18886_amd import mfmg
    case = Case(1, SPECS[name])
    rng = np.random.default_rng(5)
    r = rng.uniform(-1, 1, case.T.n)

    def results(beta, scale):
        co = mfmg.assemble_coeffs(case.tree, case.device(np.full(case.disc.n_faces, beta)),
                                  case.bc, case.theta)
        h = mfmg.build_hierarchy(co, coarsest_level=3, precision=mfmg.FP64)
        x = case.device(r * scale)
        p, st = mfmg.pcg_solve(h, x, rtol=1e-8)
        assert st["status"] == mfmg.OK
        return [v.cpu().numpy() for v in (mfmg.apply_precond(h, x),
                                          mfmg.apply_precond(h, x, transpose=True), p)]

    tiny = results(2.0 ** -1030, 2.0 ** -400)
    monkeypatch.setenv("MFMG_FUSE_BOTTOM", "0")
    for got, want in zip(tiny, results(1.0, 1.0)):
        assert np.abs(want).max() > 0.0
        assert np.array_equal(got, want * 2.0 ** 630)
