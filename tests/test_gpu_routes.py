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


@pytest.mark.parametrize("Hq,Hkv,n", [(32, 32, 8448), (32, 32, 9001)])   # 1088 and 1152 units, 1024 workgroups resident
def test_scan_just_past_the_residency(Hq, Hkv, n):
    """16-bit tiles: one unit per workgroup, not two for half of them."""
    import paper_2602_18750_amd as H
    k = torch.randn((1, Hkv, n, 128), device=DEV).to(torch.bfloat16)
    q, s = torch.randn((1, Hq, 128), device=DEV).to(torch.bfloat16), H.new_importance(1, 1, n, DEV)
    units = Hkv * 2 * ((n + 511) // 512)
    assert kernel_grids(lambda: H.hill_score(q, k, s))[0][0] == units


def _step_launches(B, Hq, Hkv, n, rows="token", streamed=True, **kw):
    """Launches of a (non-reset) step; the keys of one sequence serve the batch."""
    import paper_2602_18750_amd as H
    k = torch.randn((1, Hkv, n, 128), device=DEV).to(torch.bfloat16).expand(B, -1, -1, -1)
    q = torch.randn((B, Hq, 128), device=DEV).to(torch.bfloat16)
    R = 1 if rows == "token" else Hkv
    s, st = H.new_importance(B, R, n, DEV), H.new_stream_state(B, R, DEV) if streamed else None
    return len(kernel_grids(lambda: H.hill_step(q, k, k, s, n // 10, granularity=rows, stream_state=st, **kw)))


@pytest.mark.parametrize("B,Hq,Hkv,n,rows,refine", [
    (1, 8, 8, 32768, "kvhead", False),     # 262144 tokens in rows of one KV head each
    (8, 8, 8, 4097, "kvhead", True),       # one token per row more
    (4, 8, 1, 65536, "token", False),      # a token row of the only KV head
    (6, 16, 8, 32768, "token", False),     # 196608 tokens in rows that several KV heads walk
    (7, 16, 8, 32768, "token", True),
])
def test_streamed_selection_limit(B, Hq, Hkv, n, rows, refine):
    """A streamed step is scan, update, select and merge (so few heads need no
    statistics launch); past the limits the refine pass is among them."""
    assert _step_launches(B, Hq, Hkv, n, rows) == 4 + refine


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
