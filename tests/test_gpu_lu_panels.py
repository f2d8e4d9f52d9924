"""mfg_lu_factor at the edges of its sub-panel kernels.

A panel's kernel is picked by its height (512, 1024, 2048, 4096 rows) and the
rows' alignment; sizes sit on both sides of each line and leave partial last
panels.  Aligned and unaligned rows run the same operations in the same
order, so their factors are bitwise equal; P A = L U is held to the bound of
FP32 elimination.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1803_04014_amd as mfg
import workloads
from gpu_util import DEV, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def factor(A, lda, offset):
    n = A.shape[0]
    buf = torch.full((offset + n * lda,), float("nan"), device=DEV)
    V = buf.as_strided((n, n), (lda, 1), offset)
    V.copy_(torch.from_numpy(A))
    ipiv, info = mfg.lu_factor(V, "f32")
    return V.contiguous(), ipiv, info


@pytest.mark.parametrize("n", [1, 7, 33, 95, 512, 513, 1024, 1030, 2048, 2051, 4097])
def test_factors_at_any_height_and_alignment(n):
    A = workloads.normal(4000 + n, [(n, n)])[0].astype(np.float32)
    zero = None
    if n in (95, 1030, 2051):  # a column without a pivot: passed over and reported
        zero = n // 2
        A[:, zero] = 0.0
    LU, ipiv, info = factor(A, -(-n // 4) * 4, 0)
    assert info == (0 if zero is None else zero + 1)
    for lda, offset in ((n + 1, 0), (-(-n // 4) * 4, 1)):
        LU2, ipiv2, info2 = factor(A, lda, offset)
        assert torch.equal(LU.view(torch.int32), LU2.view(torch.int32)) and torch.equal(ipiv, ipiv2) and info == info2
    piv = host(ipiv).astype(np.int64)
    assert np.all(piv >= np.arange(n)) and np.all(piv < n)
    L = torch.tril(LU.double(), -1)
    assert float(L.abs().max()) <= 1.0
    L += torch.eye(n, dtype=torch.float64, device=DEV)
    U = torch.triu(LU.double())
    PA = torch.from_numpy(oracle.apply_pivots(piv, A).astype(np.float64)).to(DEV)
    err, scale = float((PA - L @ U).abs().max()), float((L.abs() @ U.abs()).max())
    assert err <= 4 * n * 2.0 ** -24 * scale, (err, scale)


@pytest.mark.parametrize("n,nrhs,lda", [(1, 1, 1), (63, 2, 64), (64, 1, 64), (65, 3, 67), (200, 1, 200), (513, 5, 513),
                                        (129, 2731, 132), (100, 5003, 100), (1030, 1, 1032)])
def test_substitution_at_block_edges(n, nrhs, lda):
    """Both substitutions in one chain of blocks: partial last blocks,
    unaligned rows, one and (from 8192 wavefronts) four right-hand sides per
    wavefront, the last of them partly filled.  The factors are taken as they
    are, so the reference is their FP64 solve; FP32 substitution is backward
    stable row by row: |L U x - b| <= 2 n u |L| |U| |x| to first order,
    held to twice that."""
    gen = torch.Generator(device=DEV).manual_seed(n + nrhs)
    A = torch.randn((n, n), device=DEV, generator=gen)
    V = torch.full((n, lda), float("nan"), device=DEV)[:, :n]
    V.copy_(A)
    ipiv, info = mfg.lu_factor(V, "f32")
    assert info == 0
    B = torch.randn((n, nrhs), device=DEV, generator=gen)
    X = B.clone()
    mfg.lu_solve(V, ipiv, X)
    L = torch.tril(V.double(), -1) + torch.eye(n, dtype=torch.float64, device=DEV)
    U = torch.triu(V.double())
    PB = torch.from_numpy(oracle.apply_pivots(host(ipiv).astype(np.int64), host(B)).astype(np.float64)).to(DEV)
    bound = 4 * (n + 1) * 2.0 ** -24 * (L.abs() @ (U.abs() @ X.double().abs()))
    assert bool(((L @ (U @ X.double()) - PB).abs() <= bound).all())
    again = B.clone()
    mfg.lu_solve(V, ipiv, again)
    assert torch.equal(X, again)
    one = B[:, -1:].clone()  # any grouping of right-hand sides runs the same operations
    mfg.lu_solve(V, ipiv, one)
    assert torch.equal(one, X[:, -1:])
