"""Device memory that the library gives back to the driver."""

import pytest

import problems
from gpu_fixtures import Case

pytestmark = pytest.mark.gpu

SMALL = 64 << 20  # what the driver may take besides (code, events)


def test_profile_buffers_are_not_kept():
    """The streaming copy's two 1 GiB buffers."""
    import torch
    from paper_2604_18886_amd import mfmg
    h = Case(1, problems.uniform_spec(4)).gpu_hierarchy()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    mfmg.profile(h, mfmg.PROFILE_COPY, reps=2)
    assert torch.cuda.mem_get_info()[0] >= before - SMALL


def test_release_memory():
    """What destroyed objects leave goes back on request, and objects made
    afterwards give the same results."""
    import torch
    from paper_2604_18886_amd import mfmg
    case = Case(2, problems.config_spec(2, 5, 7))

    def solve():
        h = case.gpu_hierarchy(precision=mfmg.MIXED)
        return mfmg.pcg_solve(h, case.device(case.rhs), rtol=1e-10)[0].cpu()

    mfmg.release_memory()
    first = solve()
    torch.cuda.synchronize()
    kept = torch.cuda.mem_get_info()[0]
    mfmg.release_memory()
    assert torch.cuda.mem_get_info()[0] >= kept + 100 * case.T.n
    assert torch.equal(solve(), first)
