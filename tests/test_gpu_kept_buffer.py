"""The device buffer kept between runs: every allocation of the library can
give it back when memory is short."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_allocation_can_give_the_kept_buffer_back():
    csrc = os.path.join(ROOT, "paper_2608_10075_amd", "csrc")
    raw = [(f, line.strip()) for f in sorted(os.listdir(csrc)) for line in open(os.path.join(csrc, f))
           if re.search(r"\bhipMalloc\w*\(", line) and not line.lstrip().startswith("//")]
    # device_malloc's own two calls
    assert [f for f, _ in raw] == ["twa_run.hip", "twa_run.hip"], raw
