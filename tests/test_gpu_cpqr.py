"""Row IDs below tol = 1e-7 (column-pivoted Householder QR, one launch per
pivot): every level's ID on grids whose proxy matrices cover the step
kernel's row lengths (up to and beyond 8 x 256 columns) and the
interpolation's ranks (up to 64, 128, 256, 512 and beyond).

Tolerance: the pivoting stops once every residual row has norm at most
tol ||A||_F, so the residual of the m - k other rows is at most
sqrt(m - k) tol ||A||_F; rounding adds about 1e-13 ||A||_F.  Exact ties of the
symmetric boxes leave the pivots and the rank open by a few, so the pivots
are checked for what they are: each has the largest residual norm of its step.
"""
import numpy as np
import pytest

from oracle import hbs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf,order,tol,width,kh", [
    (10, 5, 4, 1e-8, 1, 0.5), (16, 8, 4, 1e-10, 1, 0.3), (48, 6, 6, 1e-9, 2, 0.6), (56, 7, 10, 1e-10, 3, 0.4),
    (64, 8, 10, 1e-10, 3, 0.5), (128, 8, 10, 1e-10, 3, 0.5), (128, 8, 10, 1e-12, 3, 1.2)])
def test_every_level_is_a_valid_id(n, leaf, order, tol, width, kh):
    from paper_2007_12718_amd import lsh
    kappa = kh * n
    P = lsh.Plan(n, kappa, op_order=order, leaf=leaf, tol=tol, proxy_width=width, prec="fp64", hbs_order=order,
                 merge="schur")
    C = hbs.Compression(n, kappa, leaf, 0.5, width, order=order)  # (its tree and entries; the levels are P's)
    L, ranks = P.ranks()
    print(n, order, tol, ranks, flush=True)
    for l in range(L, 0, -1):
        J, cand, U = P.level(l)
        U = U.cpu().numpy()
        m, k = U.shape
        assert len(set(J.tolist())) == k and np.array_equal(U[J], np.eye(k))
        sx, sy = C.tree.box(l, 0)[2:]
        A = C.proxy_block(cand, hbs.proxy_ring(sx, sy, width))
        res = np.linalg.norm(A - U @ A[J])
        assert res <= (np.sqrt(max(m - k, 1)) * tol + 1e-13) * np.linalg.norm(A), (l, m, k)
        # the pivots are greedy: R = Q^H A^T from the unpivoted QR of A[J]^T; row i's residual norm before step t is
        # the norm of R[t:, i] and of what is left at the end
        fro = np.linalg.norm(A)
        Q = np.linalg.qr(A[J].T)[0]
        R = Q.conj().T @ A.T
        left = np.sum(np.abs(A.T - Q @ R) ** 2, axis=0)
        tail = np.sqrt(np.cumsum((np.abs(R) ** 2)[::-1], axis=0)[::-1] + left)
        tail[:, J] = np.sqrt(np.cumsum((np.abs(np.triu(R[:, J])) ** 2)[::-1], axis=0)[::-1])
        d = np.abs(np.diag(R[:, J]))
        assert np.all(d >= tail.max(axis=1) - 1e-13 * fro), (l, m, k)
        assert d.min() > tol * fro - 1e-13 * fro and np.sqrt(left.max()) <= tol * fro + 1e-13 * fro, (l, m, k)


def test_plans_repeat_bit_for_bit():
    """More rows (1396) than workgroups fit the device at once, so that the launch in which the pivoting stops still
    starts workgroups after the stop is stored: the same pivots and interpolation every time."""
    import torch
    from paper_2007_12718_amd import lsh
    o = dict(op_order=10, leaf=8, tol=1e-10, proxy_width=3, prec="fp64", hbs_order=10, merge="schur")
    ref = None
    for _ in range(3):
        P = lsh.Plan(128, 0.5 * 128, **o)
        L = P.ranks()[0]
        got = [P.level(l) for l in range(1, L + 1)]
        if ref is None:
            ref = got
        for (J, _, U), (Jr, _, Ur) in zip(got, ref):
            assert np.array_equal(J, Jr) and torch.equal(U, Ur)
        P.close()


def test_the_grids_above_reach_every_template():
    """Ranks for each interpolation kernel and row lengths for each step kernel, among two of the grids above."""
    from paper_2007_12718_amd import lsh
    ranks, cols = set(), set()
    for n, leaf, order, tol, width, kh in [(48, 6, 6, 1e-9, 2, 0.6), (128, 8, 10, 1e-12, 3, 1.2)]:
        P = lsh.Plan(n, kh * n, op_order=order, leaf=leaf, tol=tol, proxy_width=width, prec="fp64", hbs_order=order,
                     merge="schur")
        L, r = P.ranks()
        ranks |= set(r[1:])
        for l in range(1, L + 1):
            sx, sy = hbs.Compression(n, kh * n, leaf, 0.5, width, order=order).tree.box(l, 0)[2:]
            cols.add(2 * len(hbs.proxy_ring(sx, sy, width)))
    for lo, hi in [(0, 64), (64, 128), (128, 256), (256, 512), (512, 1 << 30)]:
        assert any(lo < k <= hi for k in ranks), (lo, hi, ranks)
    # (a step of column j sees the rows from j on: the longest row passes every shorter class as j advances)
    assert max(cols) > 2048, cols
