"""The row IDs' scratch sizes, which size a plan's workspace from bounds on the
row counts: a smaller row ID never needs more than a larger one (host only)."""
import ctypes

import pytest


@pytest.mark.parametrize("name", ["rowid_bp_ws", "rowid_gram_ws", "rowid_cpqr_ws"])
def test_sizes_do_not_fall_with_the_row_count(name):
    from paper_2007_12718_amd import lsh
    f = getattr(lsh.lib(), f"_ZN3lsh{len(name)}{name}Ei")
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_int]
    sizes = [f(m) for m in range(1, 4097)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
