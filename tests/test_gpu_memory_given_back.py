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
