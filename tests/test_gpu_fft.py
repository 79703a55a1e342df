"""The FFT operator at every transform length (M = r 2^k, r = 1, 3, 5, from
M >= 2n), for one and for several vectors (whole and partial groups of a
launch), against numpy's FFT of the same circulant.

Tolerance: an FFT pair of length M^2 in FP64 has a relative error of a few
2^-53 log2(M^2) in the 2-norm, below 1e-14 here; the largest entry's error
relative to the largest value is within a few times that: 1e-13.  The kernel
entries themselves (two libraries' Bessel functions) agree to 1e-13.
"""
import numpy as np
import pytest
from scipy import special

from oracle import quadrature as quad

pytestmark = pytest.mark.gpu


def cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def spectrum(n, kappa, order):
    """Transform of the 2n x 2n circulant of K, from one quadrant of its offsets."""
    d = np.arange(n)
    r = np.hypot(d[:, None], d[None, :]) / n
    K = np.zeros((n, n), complex)
    K[r > 0] = 0.25j * special.hankel1(0, kappa * r[r > 0])
    for (dx, dy), t in quad.correction_weights(order, kappa / n).items():
        if 0 <= dx < n and 0 <= dy < n:
            K[dy, dx] += t
    C = np.zeros((2 * n, 2 * n), complex)
    C[:n, :n] = K
    C[n + 1:, :n] = K[:0:-1, :]
    C[:n, n + 1:] = K[:, :0:-1]
    C[n + 1:, n + 1:] = K[:0:-1, :0:-1]
    return np.fft.fft2(C / n ** 2)


@pytest.mark.parametrize("n,leaf,nrhs", [
    (4, 2, 1), (32, 8, 3), (36, 9, 2), (40, 5, 1), (44, 11, 9), (56, 7, 2), (64, 8, 8), (80, 5, 1), (88, 11, 3),
    (96, 6, 11), (128, 8, 2), (160, 5, 1), (192, 6, 3), (256, 8, 10), (320, 5, 1), (384, 6, 2), (448, 7, 1),
    (512, 8, 9), (640, 5, 3), (768, 6, 1), (1024, 8, 3), (1280, 5, 1), (1536, 6, 1), (2048, 8, 1)])
def test_operator_at_every_length(n, leaf, nrhs):
    from paper_2007_12718_amd import lsh
    order, kappa = (4, 6, 8, 10)[n % 3], 0.3 * n
    print(n, leaf, nrhs, flush=True)
    P = lsh.Plan(n, kappa, op_order=order, leaf=leaf, tol=3e-2, proxy_width=1, prec="fp32")
    rng = np.random.default_rng(n)
    x = rng.standard_normal((nrhs, n, n)) + 1j * rng.standard_normal((nrhs, n, n))
    b = rng.uniform(-1, 1, (n, n))
    khat = spectrum(n, kappa, order)
    ref = np.stack([np.fft.ifft2(khat * np.fft.fft2(v, s=(2 * n, 2 * n)))[:n, :n] for v in x])
    out = P.apply_operator(None, cuda(x)).cpu().numpy()
    assert np.abs(out - ref).max() <= 2e-13 * np.abs(ref).max()
    A = x + kappa ** 2 * b * ref
    xc = cuda(x)
    y = P.apply_operator(cuda(b), xc)
    assert np.abs(y.cpu().numpy() - A).max() <= 2e-13 * np.abs(A).max()
    P.apply_operator(cuda(b), xc, out=xc)  # in place: the same bits
    assert np.array_equal(xc.cpu().numpy(), y.cpu().numpy())
