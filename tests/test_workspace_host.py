"""Workspace sizes of the device entry points (no GPU needed). A program that
sized its memory once, a server with a fixed budget and the allocation-free
entry point with its fixed 256 MiB accept a problem by its size, so a plan that
grows refuses what was accepted: the sizes below are upper limits."""
import pytest

import paper_1408_1664_amd as bn

LIMITS = [  # n, d, m, precision, bytes
    (2, 1, 0, "fp32", 32000), (5, 4, 0, "fp64", 33792), (8, 7, 100, "fp32", 79616),
    (10, 9, 0, "fp64", 259840), (11, 5, 300, "fp32", 366592), (12, 11, 0, "fp32", 1014272),
    (12, 3, 200, "fp64", 402432), (13, 12, 0, "fp32", 2132736), (13, 4, 700, "fp64", 1019136),
    (14, 3, 100, "fp32", 1070080), (16, 3, 1000, "fp32", 4187904),
    (20, 4, 1000, "fp64", 128367104), (22, 3, 2000, "fp32", 313731328),
    (25, 4, 2000, "fp64", 4928549632), (30, 3, 500, "fp32", 105287172608)]


@pytest.mark.parametrize("n,d,m,precision,limit", LIMITS)
def test_workspace_does_not_grow(n, d, m, precision, limit):
    assert bn.workspace_bytes(n, d, m, precision) <= limit


@pytest.mark.parametrize("n,d,m,precision", [(20, 4, 2092966, "fp32"), (20, 3, 1855869, "fp64"),
                                             (13, 12, 3198833, "fp32")])
def test_largest_problems_without_allocation(n, d, m, precision):
    assert bn.workspace_bytes(n, d, m, precision) <= bn.NOALLOC_MAX_BYTES
