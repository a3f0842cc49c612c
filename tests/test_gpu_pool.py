"""Device memory handed from destroyed objects to new ones: results do not
depend on what a block held before, on the size it is taken for or on the
thread and stream that use it."""

import threading

import numpy as np
import pytest

import problems
from gpu_fixtures import Case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cases():
    return [Case(3, problems.config_spec(3, 4, 6)), Case(2, problems.config_spec(2, 4, 6)),
            Case(1, problems.uniform_spec(4))]


def _results(case, precision):
    from paper_2604_18886_amd import mfmg
    h = case.gpu_hierarchy(precision=precision)
    p, _ = mfmg.pcg_solve(h, case.device(case.rhs), rtol=1e-10)
    g = case.device(np.where(case.disc.active, 1e-3, 0.0))
    lam, grad, _ = mfmg.pcg_solve_adjoint(h, p, g, rtol=1e-8)
    return [x.cpu().numpy() for x in (p, lam, grad)]


def test_rebuilt_objects_reproduce(cases):
    """The same bits whatever was built and destroyed before."""
    first = {(i, pr): _results(c, pr) for i, c in enumerate(cases) for pr in (0, 1)}
    for i, pr in list(first) + list(first)[::-1]:
        for a, b in zip(_results(cases[i], pr), first[i, pr]):
            assert np.array_equal(a, b)


def test_threads_and_streams(cases):
    """Threads that build, solve and destroy on streams of their own."""
    import torch
    want = [_results(c, 1) for c in cases]
    bad = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    if not all(np.array_equal(a, b)
                               for a, b in zip(_results(cases[i], 1), want[i])):
                        bad.append(i)
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # noqa: BLE001
            bad.append(repr(e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
