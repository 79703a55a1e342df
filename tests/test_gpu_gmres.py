"""The Krylov vectors' kernels: residual histories against a dense FP64 GMRES, on grids around one workgroup's piece."""
import numpy as np
import pytest
import torch

from paper_2007_12718_amd import lsh

pytestmark = pytest.mark.gpu


def _gmres_history(A, f, steps):
    """|f - A x_k| / |f| of the smallest residual over the k-th Krylov space, by an orthonormal basis from QR."""
    hist = [1.0]
    Q = [f / np.linalg.norm(f)]
    for _ in range(steps):
        w = A @ Q[-1]
        for _ in range(2):
            for q in Q:
                w = w - np.vdot(q, w) * q
        B = A @ np.stack(Q, axis=1)
        x, *_ = np.linalg.lstsq(B, f, rcond=None)
        hist.append(np.linalg.norm(f - B @ x) / np.linalg.norm(f))
        Q.append(w / np.linalg.norm(w))
    return np.array(hist)


# 36 and 100 nodes: less than a wavefront, less than a workgroup
@pytest.mark.parametrize("n", [6, 10])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_history_equals_a_dense_gmres(n, nrhs):
    rng = np.random.default_rng(n)
    kappa = 2 * np.pi
    b = torch.from_numpy(rng.uniform(0.2, 1.0, (n, n))).cuda()
    P, F = lsh.build(n, kappa, b, op_order=4, leaf=n // 2, tol=1e-8, prec="fp64")
    u = torch.from_numpy(rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n))).cuda()
    eye = torch.eye(n * n, dtype=torch.complex128, device="cuda").reshape(n * n, n, n)
    A = P.apply_operator(b, eye).reshape(n * n, n * n).T.cpu().numpy()
    f = (-kappa ** 2 * b * u)[-1].reshape(-1).cpu().numpy()
    info = F.solve(u, tol=1e-13, maxit=12, precondition=False, want_u=False)[2]
    hist = np.array(info.history[:info.iterations + 1])
    ref = _gmres_history(A, f, len(hist) - 1)
    # both are FP64 least-squares residuals of the same space: they differ by rounding times the condition of A
    tol = 100 * len(hist) * np.linalg.cond(A) * 2.0 ** -53
    assert np.abs(hist - ref).max() <= tol, (np.abs(hist - ref).max(), tol)
    F.close()
    P.close()


# one piece of a workgroup and its neighbours (4096 = 64 x 64), several pieces, and more than the group's workgroups
# cover in one go; groups of 1, 2, 3, 8 and 9 (a second group of one)
@pytest.mark.parametrize("n,nrhs", [(64, 1), (64, 8), (48, 3), (72, 2), (72, 9), (384, 8)])
def test_a_group_solves_what_single_runs_solve(n, nrhs):
    gen = torch.Generator().manual_seed(n + nrhs)
    b = torch.full((n, n), 0.3, dtype=torch.float64).cuda()
    leaf = {64: 8, 48: 12, 72: 9, 384: 12}[n]
    P, F = lsh.build(n, 12.0, b, op_order=4, leaf=leaf, tol=1e-6, prec="fp64")
    u = torch.randn(nrhs, n, n, dtype=torch.complex128, generator=gen).cuda()
    u[nrhs // 2] *= 1e-3
    if nrhs > 2:
        u[1] = 0  # a right-hand side that never runs
    sig = F.solve(u, tol=1e-11, maxit=30, want_u=False)[0]
    for r in range(nrhs):
        one = F.solve(u[r:r + 1], tol=1e-11, maxit=30, want_u=False)[0].reshape(n, n)
        # two solutions of residual 1e-11 each; the operator is a perturbation of the identity of norm below 4
        assert (sig.reshape(nrhs, n, n)[r] - one).norm() <= 2e-11 * 10 * max(one.norm().item(), 1e-300)
    F.close()
    P.close()


# some of eight vectors run, in every position of the others' gaps; one piece of a workgroup and several
@pytest.mark.parametrize("n", [48, 160])
@pytest.mark.parametrize("running", [(0,), (7,), (3, 7), (1, 2, 6), (0, 2, 4, 5, 7)])
def test_vectors_left_in_a_group_solve_what_single_runs_solve(n, running):
    gen = torch.Generator().manual_seed(n + len(running))
    b = torch.full((n, n), 0.3, dtype=torch.float64).cuda()
    P, F = lsh.build(n, 12.0, b, op_order=4, leaf=n // 8 if n == 48 else 10, tol=1e-6, prec="fp64")
    u = torch.randn(8, n, n, dtype=torch.complex128, generator=gen).cuda()
    for r in range(8):
        if r not in running:
            u[r] = 0
    sig, _, info, rc = F.solve(u, tol=1e-11, maxit=30, want_u=False)
    assert rc == 0
    for r in range(8):
        one = F.solve(u[r:r + 1], tol=1e-11, maxit=30, want_u=False)[0].reshape(n, n)
        assert (sig.reshape(8, n, n)[r] - one).norm() <= 2e-11 * 10 * max(one.norm().item(), 1e-300)
    F.close()
    P.close()


@pytest.mark.parametrize("nrhs", [1, 3])
def test_every_iteration_that_the_interface_admits(nrhs):
    """200 iterations (LSH_MAX_ITERS) without a restart, on a problem that needs more."""
    n, kappa = 24, 60.0
    rng = np.random.default_rng(0)
    b = torch.from_numpy(rng.uniform(0.2, 1.0, (n, n))).cuda()
    P, F = lsh.build(n, kappa, b, op_order=4, leaf=12, tol=1e-8, prec="fp64")
    u = torch.from_numpy(rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n))).cuda()
    eye = torch.eye(n * n, dtype=torch.complex128, device="cuda").reshape(n * n, n, n)
    A = P.apply_operator(b, eye).reshape(n * n, n * n).T.cpu().numpy()
    f = (-kappa ** 2 * b * u)[-1].reshape(-1).cpu().numpy()
    sig, _, info, rc = F.solve(u, tol=1e-13, maxit=200, precondition=False, want_u=False)
    assert rc == 1 and info.iterations == 200
    hist = np.array(info.history[:201])
    ref = _gmres_history(A, f, 200)
    tol = 100 * len(hist) * np.linalg.cond(A) * 2.0 ** -53  # (as above)
    assert np.abs(hist - ref).max() <= tol, (np.abs(hist - ref).max(), tol)
    last = sig.reshape(nrhs, -1)[-1].cpu().numpy()
    assert abs(np.linalg.norm(f - A @ last) / np.linalg.norm(f) - ref[-1]) <= tol
    F.close()
    P.close()
