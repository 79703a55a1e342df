"""The one-launch apply levels, for M and M^T, against the batched products:
every eligible level fused against none, over right-hand-side counts that
leave whole and partial groups (groups of 4, 2 and 1), both precisions, leaf
sizes that give odd skeletons, and row lengths on both sides of the 16- and
32-entry lane layouts.

Tolerance: the two forms sum the same products in another order; an apply is a
chain of a few dozen products of length at most 2c, so they agree to about
sqrt(2c) u per product in the working precision u, amplified by the factor's
condition: 2e-5 in FP32, 1e-12 in FP64 relative to the largest entry.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("prec,tol", [("fp32", 2e-5), ("fp64", 1e-12)])
@pytest.mark.parametrize("n,leaf,kh", [(16, 4, 0.5), (40, 5, 0.6), (64, 8, 0.3), (112, 7, 0.5), (192, 6, 0.62)])
def test_fused_levels_match_batched_products(n, leaf, kh, prec, tol):
    import torch
    from paper_2007_12718_amd import lsh
    rng = np.random.default_rng(n)
    b = cuda(synth.bumps(n, rng))
    P = lsh.Plan(n, kh * n, op_order=4, leaf=leaf, tol=1e-4, proxy_width=2, prec=prec, merge="lowrank")
    F = lsh.Factor(P, b, transpose=True)
    try:
        for nrhs in (1, 2, 3, 4, 7, 9):
            x = cuda(rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n)))
            for tr in (False, True):
                lsh.apply_fused_levels(0)
                ref = F.apply_precond(x, transpose=tr)
                for least in (1, -1):
                    lsh.apply_fused_levels(least)
                    y = F.apply_precond(x, transpose=tr)
                    err = float((y - ref).abs().max() / ref.abs().max())
                    assert err <= tol, (nrhs, tr, least, err)
                    one = F.apply_precond(x[nrhs - 1:], transpose=tr)
                    assert float((one[0] - ref[nrhs - 1]).abs().max() / ref.abs().max()) <= tol
    finally:
        lsh.apply_fused_levels(-1)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,leaf,kh", [(16, 4, 0.5), (40, 5, 0.6), (64, 8, 0.3), (112, 7, 0.5), (192, 6, 0.62)])
def test_the_comparison_above_runs_the_fused_kernels(n, leaf, kh, prec):
    """Its thresholds launch what it compares: both one-launch passes of either direction, or none of them."""
    import torch
    from paper_2007_12718_amd import lsh
    b = cuda(synth.bumps(n, np.random.default_rng(n)))
    P = lsh.Plan(n, kh * n, op_order=4, leaf=leaf, tol=1e-4, proxy_width=2, prec=prec, merge="lowrank")
    F = lsh.Factor(P, b, transpose=True)
    x = torch.ones((3, n, n), dtype=torch.complex128, device="cuda")
    F.apply_precond(x, transpose=True)  # (the first one builds the transposed copies)
    names = [f"level_{p}_{'f32' if prec == 'fp32' else 'f64'}" for p in ("up", "down", "tup", "tdown")]
    try:
        for least in (1, -1, 0):
            for tr in (False, True):
                lsh.apply_fused_levels(least)
                lsh.lsh_profile_enable(True)
                F.apply_precond(x, transpose=tr)
                ran = [lsh.lsh_profile_query(k)[0] > 0 for k in names]
                lsh.lsh_profile_enable(False)
                want = [not tr, not tr, tr, tr] if least else [False] * 4
                assert ran == want, (least, tr, ran)
    finally:
        lsh.lsh_profile_enable(False)
        lsh.apply_fused_levels(-1)
