"""The matrix products' staging: every operand order at the edges of the tiles, and nothing read from outside."""
import ctypes

import pytest
import torch

from paper_2007_12718_amd import lsh

pytestmark = pytest.mark.gpu

OPS = {0: lambda X: X, 1: lambda X: X.transpose(-1, -2), 2: lambda X: X.conj().transpose(-1, -2), 3: lambda X: X.conj()}


def _op(X, op):
    return OPS[op](X).resolve_conj()


def _product(A, B, opA=0, opB=0):
    """op(A) op(B) of (batch, rows, cols) views that may be parts of wider arrays."""
    M, K = A.shape[-2:] if opA in (0, 3) else A.shape[:-3:-1]
    N = B.shape[-1] if opB in (0, 3) else B.shape[-2]
    C = torch.empty(A.shape[0], M, N, dtype=A.dtype, device="cuda")
    prec = lsh.LSH_FP64 if A.dtype == torch.complex128 else lsh.LSH_FP32
    two = ctypes.c_double * 2
    p = lambda X: ctypes.c_void_p(X.data_ptr())
    st = lambda X: (X.stride(1), X.stride(0))
    lsh._check(lsh.lib().lsh_dev_gemm(prec, M, N, K, two(1, 0), p(A), *st(A), opA, p(B), *st(B), opB, two(0, 0),
                                      None, N, 0, p(C), N, M * N, A.shape[0], lsh._stream()))
    return C


def _operand(rows, cols, op, batch, dt, gen):
    """A stored operand whose op(.) is rows x cols, inside a wider array of NaN."""
    r, c = (rows, cols) if op in (0, 3) else (cols, rows)
    wide = torch.full((batch, r + 1, c + 3), complex("nan"), dtype=dt)
    wide[:, :r, :c] = torch.randn(batch, r, c, dtype=torch.complex128, generator=gen).to(dt)
    dev = wide.cuda()
    return wide[:, :r, :c], dev[:, :r, :c]


# one below, at and above the 16-, 32- and 64-deep K tiles and the 64- and 128-wide tiles
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (63, 65, 15), (64, 64, 64), (65, 63, 33), (128, 129, 31), (127, 128, 65)])
def test_every_order_at_the_tile_edges(prec, M, N, K):
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    u = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    gen = torch.Generator().manual_seed(1000 * M + K)
    for opA in range(4):
        for opB in range(4):
            hA, A = _operand(M, K, opA, 2, dt, gen)
            hB, B = _operand(K, N, opB, 2, dt, gen)
            X, Y = _op(hA, opA).to(torch.complex128), _op(hB, opB).to(torch.complex128)
            ref = torch.stack([x @ y for x, y in zip(X, Y)])
            # a sum of 4 K (or, by three products, 6 K) rounded terms of at most 2 |a| |b| each
            bound = 2 * (6 * K + 8) * u * torch.stack([x.abs() @ y.abs() for x, y in zip(X, Y)])
            for v in range(len(lsh.gemm_variants(prec))):
                lsh.gemm_force_variant(v)
                try:
                    C = _product(A, B, opA, opB).cpu()
                finally:
                    lsh.gemm_force_variant(-1)
                assert ((C.to(torch.complex128) - ref).abs() <= bound).all(), (opA, opB, v)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_an_infinity_stays_in_its_row(prec):
    """What lies outside a tile is read as the first element and dropped, whatever that element is."""
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    A = torch.ones(1, 70, 37, dtype=dt)
    A[0, 0, 0] = complex("inf")
    B = torch.ones(1, 37, 70, dtype=dt)
    C = _product(A.cuda(), B.cuda()).cpu()[0]
    assert not torch.isfinite(torch.view_as_real(C[0])).all()
    assert (C[1:] == 37).all()


@pytest.mark.parametrize("order,name", [(64, "cgemm_f64_32x32k32"), (1600, "cgemm_f64_32x32k32"),
                                        (2048, "cgemm_f64_64x64k32"), (4160, "cgemm_f64_64x64k32"),
                                        (6000, "cgemm_f64_64x64k32")])
def test_fp64_tile_by_rounds(order, name):
    """Without a table: the small tile for one round or clearly shorter ones, the large one for many full rounds."""
    import torch
    from paper_2007_12718_amd import lsh
    A = torch.randn(1, order, 8, dtype=torch.complex128, device="cuda")
    B = torch.randn(1, 8, order, dtype=torch.complex128, device="cuda")
    lsh.gemm_table_clear()
    try:
        lsh.lsh_profile_enable(True)
        C = lsh.dev_gemm(A, B)
        names = lsh.lsh_profile_names()
    finally:
        lsh.lsh_profile_enable(False)
        lsh.gemm_table_load(lsh.GEMM_TABLE)
    assert [k for k in names if k.startswith("cgemm")] == [name]
    # sums of eight products of normal numbers: below 8 * 16 * 2^-53 times the largest
    assert float((C - A @ B).abs().max()) <= 1e-13


@pytest.mark.parametrize("M,N,K,batch,name", [
    (256, 256, 128, 64, "cgemm_f32_128x64"), (300, 1000, 64, 32, "cgemm_f32_64x64"),
    (76, 1243, 10, 64, "cgemm_f32_64x64"), (64, 64, 64, 8, "cgemm_f32_64x64")])
def test_fp32_tile_by_area_and_depth(M, N, K, batch, name):
    """Without a table: the larger tile only beyond one K stage and where its edge covers no more than 64 x 64 tiles."""
    import torch
    from paper_2007_12718_amd import lsh
    A = torch.randn(batch, M, K, dtype=torch.complex64, device="cuda")
    B = torch.randn(batch, K, N, dtype=torch.complex64, device="cuda")
    lsh.gemm_table_clear()
    try:
        lsh.lsh_profile_enable(True)
        C = lsh.dev_gemm(A, B)
        names = lsh.lsh_profile_names()
    finally:
        lsh.lsh_profile_enable(False)
        lsh.gemm_table_load(lsh.GEMM_TABLE)
    assert [k for k in names if k.startswith("cgemm")] == [name]
    ref = A[0].to(torch.complex128) @ B[0].to(torch.complex128)
    # 3 K + 4 roundings of a sum of K products, three real products to a complex one
    assert float((C[0] - ref).abs().max()) <= (3 * K + 4) * 2.0 ** -24 * float(ref.abs().max())
