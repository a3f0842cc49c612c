"""As test_gpu_cache_policy, for the transposed cycle and the adjoint solve:
their half-sweeps, first half-sweeps, restriction and operator have streamed
forms of their own, which change no arithmetic."""

import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r'''
import sys
import numpy as np
sys.path.insert(0, {root!r})
sys.path.insert(0, {tests!r})
from gpu_fixtures import small_cases
from paper_2604_18886_amd import mfmg
case = small_cases()["cut_sphere_5_7"]()
out = {{}}
for prec in (0, 1):
    h = case.gpu_hierarchy(precision=prec, mu=1 + prec)
    rng = np.random.default_rng(41)
    r = case.device(np.where(case.disc.active, rng.uniform(-1, 1, case.T.n), 0.0))
    out["z%d" % prec] = mfmg.apply_precond(h, r, transpose=True).cpu().numpy()
    p, _ = mfmg.pcg_solve(h, case.device(case.rhs), rtol=1e-10)
    lam, grad, st = mfmg.pcg_solve_adjoint(h, p, r, rtol=1e-10)
    out["lam%d" % prec] = lam.cpu().numpy()
    out["grad%d" % prec] = grad.cpu().numpy()
    out["it%d" % prec] = np.array([st["iters"]])
np.savez({path!r}, **out)
'''


def _run(tmp_path, stream_bytes, tag):
    path = str(tmp_path / f"{tag}.npz")
    env = dict(os.environ, MFMG_STREAM_BYTES=str(stream_bytes))
    code = CHILD.format(root=ROOT, tests=HERE, path=path)
    print(f"  child MFMG_STREAM_BYTES={stream_bytes}", flush=True)
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return dict(np.load(path))


def test_streamed_levels_compute_the_same_values(tmp_path):
    every = _run(tmp_path, 0, "every_level_streamed")
    none = _run(tmp_path, 1 << 50, "no_level_streamed")
    assert set(every) == set(none)
    for key in none:
        assert np.abs(none[key]).max() > 0.0
        assert np.array_equal(every[key], none[key]), key
