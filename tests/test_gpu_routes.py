"""Which kernels a call launches, read from its captured graph: the rules that
choose between forms of one operation must depend on the call alone."""
import os
import subprocess
import sys

import pytest
import torch

from util import kernel_grids

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TESTS = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_18750_amd as H
    H.load_library()
    yield


# The scans' grids are capped at what stays resident on the chip, a number of
# each kernel's own, asked for once per process.
SCAN_GRIDS = r"""
import sys
sys.path[:0] = [%r, %r]
import torch
import paper_2602_18750_amd as H
from util import kernel_grids
k = torch.randn((1, 8, 32768, 128), device="cuda:0").to(torch.bfloat16)
for B in [int(x) for x in sys.argv[1:]]:     # a batch over one sequence's keys
    q = torch.randn((B, 32, 128), device="cuda:0").to(torch.bfloat16)
    s = H.new_importance(B, 1, 32768, "cuda:0")
    kb = k.expand(B, -1, -1, -1)
    print(B, kernel_grids(lambda: H.hill_score(q, kb, s))[0][0])
"""


def test_scan_grid_does_not_depend_on_earlier_calls():
    """Scans of 2 and 8 x 32K tokens (two kernels of different residency), each
    the first of its process once: the same grids in either order."""
    code = SCAN_GRIDS % (TESTS, os.path.dirname(TESTS))
    out = []
    for order in (["2", "8"], ["8", "2"]):
        r = subprocess.run([sys.executable, "-c", code] + order, capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stderr[-2000:]
        out.append(sorted(r.stdout.split("\n")))
    assert out[0] == out[1]
