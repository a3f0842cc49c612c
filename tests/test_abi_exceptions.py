"""Nothing throws across the C ABI: every handler of a HIP error at an entry
point is followed by one of std::bad_alloc (host vectors and the device pools'
table are allocated under most of them).  Read from the source, as a failing
host allocation cannot be had without a device to reach it."""

import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2604_18886_amd", "csrc", "mfmg.hip")


def test_hip_error_handlers_also_catch_bad_alloc():
    text = open(SRC).read()
    handlers = [m.start() for m in re.finditer(r"catch \(const HipError &", text)]
    assert len(handlers) >= 15
    for at in handlers:
        after = re.match(r"catch \(const HipError &\w+\) \{[^{}]*\} catch \(const std::bad_alloc &\)",
                         text[at:])
        line = text.count("\n", 0, at) + 1
        assert after, f"mfmg.hip:{line}: std::bad_alloc would leave the C entry"
