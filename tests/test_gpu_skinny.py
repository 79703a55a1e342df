"""Products of a matrix with a few vectors on the matrix instruction: groups against the same vectors one at a time.

With the one-launch levels off, a group of three vectors or more takes every box product through the 16-row tiles;
one vector at a time takes the per-box products through the row-streaming kernel.  The grids give matrices below one
tile, odd row lengths on both sides of the 16-deep chunks, and up to 9 x 2^l vectors on the shared matrices.

Tolerance: the two forms sum the same products in another order; an apply is a chain of a few dozen products of length
at most 2c, so they agree to about sqrt(2c) u per product in FP32, amplified by the factor's condition: 2e-5 relative to
the largest entry.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("full", [0, 1])
@pytest.mark.parametrize("n,leaf,kh", [(10, 5, 0.5), (24, 6, 0.6), (44, 11, 0.4), (96, 12, 0.5), (160, 5, 0.6)])
def test_groups_match_single_vectors(n, leaf, kh, full):
    import torch
    from paper_2007_12718_amd import lsh
    rng = np.random.default_rng(n + full)
    b = cuda(synth.bumps(n, rng))
    P = lsh.Plan(n, kh * n, op_order=4, leaf=leaf, tol=1e-4, proxy_width=2, prec="fp32", merge="lowrank",
                 full_levels=full)
    F = lsh.Factor(P, b, transpose=True)
    try:
        x = cuda(rng.standard_normal((9, n, n)) + 1j * rng.standard_normal((9, n, n)))
        for tr in (False, True):
            lsh.apply_fused_levels(0)
            ref = torch.cat([F.apply_precond(x[r:r + 1], transpose=tr) for r in range(9)])
            for least in (0, -1):
                lsh.apply_fused_levels(least)
                for nrhs in (2, 3, 5, 8, 9):
                    y = F.apply_precond(x[:nrhs], transpose=tr)
                    assert float((y - ref[:nrhs]).abs().max() / ref.abs().max()) <= 2e-5, (tr, least, nrhs)
    finally:
        lsh.apply_fused_levels(-1)
