"""Compiler resource report of the HIP kernels (no GPU needed): no kernel may
use scratch memory.  A private array that the compiler cannot keep in
registers (an indexed pick, an array captured by reference) moves the whole
per-lane state to scratch and costs the scan a factor of two, silently."""
import os

import pytest


@pytest.fixture(scope="module")
def report():
    from paper_2602_18750_amd import _build
    if not os.path.exists(_build.RESOURCES) or not os.path.exists(_build.LIB):
        _build.build()
    rows = [l.rstrip("\n").split("\t") for l in open(_build.RESOURCES) if l.strip()]
    return rows


def test_every_kernel_is_reported(report):
    names = " ".join(r[1] for r in report)
    for k in ("score_tiles_kernel", "update_attn_kernel", "topk_refine_kernel", "topk_emit_kernel",
              "merge_write_kernel", "sketch_keys_kernel", "bkp_rank_kernel", "calib_read_kernel"):
        assert k in names, k


def test_exact_groups_have_kernels_without_masks(report):
    """Groups of 1, 2, 4 and 8 heads per pass select and attend without the
    clamps and tests of a masked pass (the last template argument)."""
    for gc in (1, 2, 4, 8):
        for name in ("topk_emit_kernelILi1ELi%dELb1E" % gc, "attn_split_kernelILi1ELi%dE" % gc):
            last = {r[1].split("EEEv")[0][-3:] for r in report if name in r[1]}
            assert last == ({"Lb0", "Lb1"} if gc >= 4 else {"Lb0"}), (name, last)


def test_no_kernel_uses_scratch(report):
    bad = [(r[0], r[1], r[3]) for r in report if r[3] != "scratch=0"]
    assert not bad, bad


def test_resident_scan_workgroups(report):
    """The scans hide memory latency by the workgroups (of one wave per SIMD)
    that fit a CU together: 16-bit matrix-core 6, int8 5, int4 4."""
    want = {"KeysF16MfmaILi": 6, "KeysSketchMfma8ILi": 5, "KeysSketchMfma4ILi": 4}
    for name, n in want.items():
        got = [int(r[4].split("=")[1]) for r in report if "score_tiles_kernel" in r[1] and name in r[1]]
        assert len(got) == 2 and min(got) >= n, (name, got)
