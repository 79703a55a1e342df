"""The receiver sums and their adjoint: the kernel (i/4) H0 over its whole
argument range (both branches and their boundary), and both maps over numbers
of points and fields that meet every template and remainder.

Tolerances.  The argument kappa r carries four roundings (difference, squares
and sum, root, product), each worth up to kappa r 2^-53 of phase, on either
side, and the evaluation about 5e-16 |H0|.  The sums over N nodes add
pairwise-like rounding of 1e-13 of the largest value at these sizes.
"""
import numpy as np
import pytest
from scipy import special

from oracle import dense

pytestmark = pytest.mark.gpu


def cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("kappa", [1e-3, 3.0, 40.0, 2e3, 3e6])
def test_kernel_values_over_the_argument_range(kappa):
    """One unit node: every receiver's value is h^2 (i/4) H0(kappa r)."""
    from paper_2007_12718_amd import lsh
    n = 10
    plan = lsh.Plan(n, kappa, op_order=4, leaf=5, tol=0.0, proxy_width=1, prec="fp64")
    h = 1.0 / n
    rng = np.random.default_rng(0)
    r = np.concatenate([10.0 ** rng.uniform(-6, 1.5, 3000), 8.0 * (1 + 1e-3 * rng.uniform(-1, 1, 200)) / kappa])
    t = rng.uniform(0, 2 * np.pi, r.size)
    x0 = -0.5 + 3.5 * h
    pts = np.stack([x0 + r * np.cos(t), x0 + r * np.sin(t)], axis=1)
    sig = np.zeros((1, n, n), complex)
    sig[0, 3, 3] = 1.0
    out = plan.eval_points(cuda(sig), cuda(pts)).cpu().numpy()[0]
    rr = np.hypot(pts[:, 0] - x0, pts[:, 1] - x0)
    ref = h * h * 0.25j * special.hankel1(0, kappa * rr)
    # r itself is rounded where the point is added to the node (absolute 2^-53 of the coordinates)
    slack = kappa * (8 * rr + 2.0) * 2.0 ** -53 + kappa * 4e-16 / np.maximum(kappa * rr, 1e-300) + 2e-15
    assert np.all(np.abs(out - ref) <= slack * np.abs(ref))
    back = plan.eval_points_adjoint(cuda(np.ones((1, 1), complex)), cuda(pts[:1])).cpu().numpy()[0, 3, 3]
    assert abs(back - np.conj(ref[0])) <= slack[0] * abs(ref[0])


def test_points_on_a_node_and_at_infinity():
    """A receiver on a node has an infinite value there; one at infinity gets zero."""
    from paper_2007_12718_amd import lsh
    n = 8
    P = lsh.Plan(n, 5.0, op_order=4, leaf=4, tol=1e-3, proxy_width=1, prec="fp64")
    sig = np.zeros((1, n, n), complex)
    sig[0, 2, 3] = 1.0
    pts = np.array([[-0.5 + 3.5 / n, -0.5 + 2.5 / n], [np.inf, 0.0], [1e200, 0.0], [0.9, 0.9]])
    out = P.eval_points(cuda(sig), cuda(pts)).cpu().numpy()[0]
    assert not np.isfinite(out[0]) and out[1] == 0 and out[2] == 0 and np.isfinite(out[3]) and out[3] != 0


@pytest.mark.parametrize("n,leaf,npts,nrhs", [(8, 4, 1, 1), (40, 5, 3, 2), (64, 8, 17, 3), (96, 6, 64, 8),
                                               (112, 7, 5, 9), (384, 6, 4, 5), (40, 5, 5000, 1)])
def test_forward_and_adjoint_match_the_dense_matrix(n, leaf, npts, nrhs):
    from paper_2007_12718_amd import lsh
    kappa = 0.5 * n
    rng = np.random.default_rng(n + npts)
    t = rng.uniform(0, 2 * np.pi, npts)
    pts = np.stack([0.8 * np.cos(t), 0.8 * np.sin(t)], axis=1)
    sig = rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n))
    g = rng.standard_normal((nrhs, npts)) + 1j * rng.standard_normal((nrhs, npts))
    P = lsh.Plan(n, kappa, op_order=4, leaf=leaf, tol=1e-2, proxy_width=1, prec="fp64")
    E = dense.receiver_matrix(n, kappa, pts)
    out = P.eval_points(cuda(sig), cuda(pts)).cpu().numpy()
    ref = sig.reshape(nrhs, -1) @ E.T
    assert np.abs(out - ref).max() <= 1e-13 * np.abs(ref).max() * max(1.0, np.sqrt(n) / 8)
    back = P.eval_points_adjoint(cuda(g), cuda(pts)).cpu().numpy().reshape(nrhs, -1)
    refb = g @ E.conj()
    assert np.abs(back - refb).max() <= 1e-13 * np.abs(refb).max() * max(1.0, np.sqrt(n) / 8)


def test_calls_on_two_streams_take_turns():
    """Calls of one plan on two streams, without a wait between them, give each its own result."""
    import torch
    from paper_2007_12718_amd import lsh
    n, nrhs = 256, 8
    P = lsh.Plan(n, 100.0, op_order=4, leaf=8, tol=1e-2, proxy_width=1, prec="fp64")
    rng = np.random.default_rng(4)
    t = rng.uniform(0, 2 * np.pi, 33)
    xy = cuda(np.stack([0.8 * np.cos(t), 0.8 * np.sin(t)], axis=1))
    sig = [cuda(rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n))) for _ in range(2)]
    ref = [P.eval_points(s, xy) for s in sig]
    torch.cuda.synchronize()
    st = [torch.cuda.Stream() for _ in range(2)]
    outs = []
    for k in range(6):
        with torch.cuda.stream(st[k % 2]):
            outs.append(P.eval_points(sig[k % 2], xy))
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref[k % 2]) for k, o in enumerate(outs))


@pytest.mark.parametrize("lo,hi,tol", [(1e-8, 0.5, 3.5e-16), (0.5, 14.0, 1.7e-16), (14.0, 1e4, 5e-16)])
def test_kernel_values_to_the_last_bits(lo, hi, tol):
    """Arguments that reach the kernel exactly (kappa = 1, receivers on the axis through a node at 0).  Below 1/2 the
    logarithm may be off by one unit in the last place and the sum is rounded; up to 14 both parts are rounded once and
    the terms behind the first, at most an eighth of |H1|, three times; beyond, the stated bound."""
    mpmath = pytest.importorskip("mpmath")
    from paper_2007_12718_amd import lsh
    plan = lsh.Plan(4, 1.0, op_order=4, leaf=2, tol=0.0, proxy_width=1, prec="fp64", h=0.25, x0=-0.125, y0=-0.125)
    rng = np.random.default_rng(7)
    r = np.concatenate([lo * (hi / lo) ** rng.random(600), rng.uniform(lo, hi, 600)])
    edges = np.concatenate([np.arange(8, 16) / 16, np.arange(8, 16) / 8, np.arange(8, 57) / 4])
    r = np.concatenate([r, np.nextafter(edges, 0), np.nextafter(edges, 99)])
    r = r[(r >= lo) & (r < hi)]
    sig = np.zeros((1, 4, 4), complex)
    sig[0, 0, 0] = 16.0
    out = plan.eval_points(cuda(sig), cuda(np.stack([r, 0 * r], axis=1))).cpu().numpy()[0]
    with mpmath.workdps(30):
        for x, v in zip(r.tolist(), out.tolist()):
            ref = (1j * mpmath.besselj(0, x) - mpmath.bessely(0, x)) / 4
            assert abs(mpmath.mpc(v) - ref) <= tol * abs(ref), (x, v)


def test_calls_from_two_threads_take_turns():
    """The same from two host threads, each on its own stream."""
    import threading

    import torch
    from paper_2007_12718_amd import lsh
    n, nrhs = 256, 8
    P = lsh.Plan(n, 100.0, op_order=4, leaf=8, tol=1e-2, proxy_width=1, prec="fp64")
    rng = np.random.default_rng(5)
    t = rng.uniform(0, 2 * np.pi, 33)
    xy = cuda(np.stack([0.8 * np.cos(t), 0.8 * np.sin(t)], axis=1))
    sig = [cuda(rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n))) for _ in range(2)]
    ref = [P.eval_points(s, xy) for s in sig]
    torch.cuda.synchronize()
    outs, err = [[], []], []

    def calls(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                outs[i] = [P.eval_points(sig[i], xy) for _ in range(50)]
                torch.cuda.current_stream().synchronize()
        except Exception as e:  # (reported by the main thread)
            err.append(e)

    ths = [threading.Thread(target=calls, args=(i,)) for i in range(2)]
    for th in ths:
        th.start()
    for th in ths:
        th.join()
    assert not err, err
    for i in range(2):
        assert len(outs[i]) == 50 and all(torch.equal(o, ref[i]) for o in outs[i])


@pytest.mark.parametrize("n,leaf,npts,nrhs", [(16, 4, 1, 16), (64, 8, 3, 17), (384, 6, 9, 17), (384, 6, 9, 24)])
def test_groups_of_fields_on_the_grid(n, leaf, npts, nrhs):
    """Whole groups of eight in one launch, with a partial last one (small calls) or that one by itself."""
    from paper_2007_12718_amd import lsh
    rng = np.random.default_rng(nrhs)
    t = rng.uniform(0, 2 * np.pi, npts)
    pts = np.stack([0.8 * np.cos(t), 0.8 * np.sin(t)], axis=1)
    sig = rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n))
    g = rng.standard_normal((nrhs, npts)) + 1j * rng.standard_normal((nrhs, npts))
    P = lsh.Plan(n, 0.5 * n, op_order=4, leaf=leaf, tol=1e-2, proxy_width=1, prec="fp64")
    E = dense.receiver_matrix(n, 0.5 * n, pts)
    ref, refb = sig.reshape(nrhs, -1) @ E.T, g @ E.conj()
    out = P.eval_points(cuda(sig), cuda(pts)).cpu().numpy()
    back = P.eval_points_adjoint(cuda(g), cuda(pts)).cpu().numpy().reshape(nrhs, -1)
    tol = 1e-13 * max(1.0, np.sqrt(n) / 8)
    for r in range(nrhs):
        assert np.abs(out[r] - ref[r]).max() <= tol * np.abs(ref).max(), r
        assert np.abs(back[r] - refb[r]).max() <= tol * np.abs(refb).max(), r


@pytest.mark.parametrize("n,leaf,npts,nrhs", [(96, 6, 1, 1), (96, 6, 7, 2), (96, 6, 5, 4), (96, 6, 9, 8),
                                               (64, 8, 3, 17)])
def test_captured_calls(n, leaf, npts, nrhs):
    """Under capture the forward sums take the grid in one part, without the plan's memory: replays on new inputs,
    with eager calls between them, against the eager results."""
    import torch
    from paper_2007_12718_amd import lsh
    P = lsh.Plan(n, 0.5 * n, op_order=4, leaf=leaf, tol=1e-2, proxy_width=1, prec="fp64")
    gen = torch.Generator(device="cuda").manual_seed(npts)

    def field(*shape):
        return torch.randn(*shape, dtype=torch.complex128, device="cuda", generator=gen)

    xy = 0.6 + torch.rand(npts, 2, dtype=torch.float64, device="cuda", generator=gen)
    sig, g = field(nrhs, n, n), field(nrhs, npts)
    P.eval_points(sig, xy)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out, back = P.eval_points(sig, xy), P.eval_points_adjoint(g, xy)
    for _ in range(3):
        sig.copy_(field(nrhs, n, n))
        g.copy_(field(nrhs, npts))
        graph.replay()
        ref, refb = P.eval_points(sig, xy), P.eval_points_adjoint(g, xy)
        torch.cuda.synchronize()
        # (another order of the sum over the nodes)
        assert float((out - ref).abs().max()) <= 1e-13 * float(ref.abs().max()) * max(1.0, n ** 0.5 / 8)
        assert torch.equal(back, refb)
