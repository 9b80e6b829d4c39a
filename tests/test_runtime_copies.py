"""Host check: the library makes no strided copies of the runtime's (2-D, 3-D).
Into ordinary host memory they leave the data out, without an error, in a
process that a profiler records; strided data is gathered by kernels."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1705_04702_amd", "csrc")


def test_no_strided_copies():
    found = [f for f in sorted(os.listdir(CSRC)) if re.search(r"hipMemcpy[23]D", open(os.path.join(CSRC, f)).read())]
    assert found == []
