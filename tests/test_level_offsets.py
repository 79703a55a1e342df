"""The one-launch apply levels reach the second sibling block by unsigned
32-bit byte offsets from the first: the rule that admits a level admits only
distances whose offsets are the distances (host only)."""
import ctypes

import pytest


@pytest.mark.parametrize("size", [8, 16])
def test_admitted_distances_survive_the_offsets(size):
    from paper_2007_12718_amd import lsh
    fit = lsh.lib()._ZN3lsh17level_offsets_fitEl
    fit.restype, fit.argtypes = ctypes.c_bool, [ctypes.c_long]
    last = (65536 // (6 * size)) ** 2 - 1  # last entry of the largest block whose vectors fit the LDS
    for d in [-(1 << 27), -4096, -1, 0, 1, 90 * 90, 1 << 20, (1 << 27) - 1, 1 << 27, (1 << 27) + 1, 1 << 28, 1 << 40]:
        if fit(d):
            assert ((d + last) * size) % (1 << 32) == (d + last) * size and (d * size) % (1 << 32) == d * size, d
    assert fit(0) and fit(90 * 90) and fit(1 << 27)
