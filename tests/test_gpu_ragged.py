"""Ragged M, N, K on the kernels the library picks by default.

The 16-bit kernels differ only in how output tiles are assigned to
workgroups, so the default choice at any size is held bitwise to the simple
kernel (configuration 0), whose parity with the oracle test_gpu_gemm.py
checks.  Sizes sit at the edges of the tiles, of the 64-deep stages and of
the 16-byte pieces (K % 8, N % 8); NaN fills the operands' padding and, under
beta = 0, C.
"""
import pytest
import torch

import paper_1803_04014_amd as mfg
from gpu_util import DEV, need_gpu

pytestmark = pytest.mark.gpu

PLANES = {"f16": (1, 1), "bf16": (1, 1), "refine_a": (2, 1), "split3": (2, 2), "split4": (2, 2), "bf16_split3": (2, 2)}
# smallest, tile and stage edges, one straddling piece per remainder, skinny, then one per larger tile
SHAPES = [(1, 1, 1), (32, 64, 64), (33, 65, 65), (65, 7, 200), (64, 130, 63), (129, 129, 129), (31, 600, 1003), (600, 33, 518),
          (200, 333, 257), (777, 1234, 330), (1500, 1501, 396), (2000, 4001, 133), (2999, 3001, 2003)]


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def plane_matrix(rows, cols, planes, dtype, gen):
    """`planes` stacked rows x cols planes, 16-byte rows, NaN beyond each row's last column."""
    ld = -(-cols // 8) * 8
    buf = torch.full((planes * rows, ld), float("nan"), dtype=dtype, device=DEV)
    buf[:, :cols] = torch.rand((planes * rows, cols), device=DEV, generator=gen).mul_(2).sub_(1).to(dtype)
    return buf.as_strided((rows, cols), (ld, 1))


@pytest.mark.parametrize("mode", sorted(PLANES))
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_default_choice_is_bitwise_the_simple_kernel(mode, shape):
    M, N, K = shape
    gen = torch.Generator(device=DEV).manual_seed(M * 7 + N * 3 + K)
    dtype = torch.bfloat16 if mode.startswith("bf16") else torch.float16
    A = plane_matrix(M, K, PLANES[mode][0], dtype, gen)
    B = plane_matrix(K, N, PLANES[mode][1], dtype, gen)
    C0 = torch.rand((M, N), device=DEV, generator=gen)
    for alpha, beta in ((1.0, 0.0), (1.25, -0.5)):
        out = []
        for config in (0, -1):
            C = torch.full((M, N), float("nan"), device=DEV) if beta == 0.0 else C0.clone()
            mfg.gemm(A, B, C, alpha, beta, mode=mode, preconverted=True, config=config)
            out.append(C)
        assert torch.isfinite(out[0]).all()
        assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32)), (alpha, beta)


@pytest.mark.parametrize("shape", [(33, 40, 24), (40, 56, 48), (64, 64, 64), (48, 120, 88), (200, 72, 130)], ids=str)
@pytest.mark.parametrize("mode", ["f16", "split3"])
def test_batched_entries_are_bitwise_solo(mode, shape):
    M, N, K = shape
    count = 37
    gen = torch.Generator(device=DEV).manual_seed(count)
    p = PLANES[mode]
    lda, ldb = -(-K // 8) * 8, -(-N // 8) * 8
    A = torch.rand((count, p[0] * M, lda), device=DEV, generator=gen).half()
    B = torch.rand((count, p[1] * K, ldb), device=DEV, generator=gen).half()
    C = torch.full((count, M, N), float("nan"), device=DEV)
    mfg.gemm_batched(A[:, :M, :K], B[:, :K, :N], C, mode=mode, preconverted=True)
    for i in range(count):
        solo = torch.empty((M, N), device=DEV)
        mfg.gemm(A[i, :M, :K], B[i, :K, :N], solo, mode=mode, preconverted=True, config=0)
        assert torch.equal(C[i].view(torch.int32), solo.view(torch.int32)), i


# FP32: edges of the 64 / 128 tiles and of the 32-deep stages, rows 16-byte aligned and not
F32_SHAPES = [(1, 1, 1), (33, 32, 33), (64, 64, 64), (65, 130, 31), (129, 63, 100), (200, 333, 257), (127, 1100, 40),
              (700, 900, 515), (1300, 1500, 260), (2050, 2052, 132)]


@pytest.mark.parametrize("aligned", [True, False], ids=["aligned", "unaligned"])
@pytest.mark.parametrize("shape", F32_SHAPES, ids=str)
def test_f32_default_choice_is_bitwise_the_simple_kernel(shape, aligned):
    M, N, K = shape
    gen = torch.Generator(device=DEV).manual_seed(M + N + K)

    def matrix(rows, cols):
        ld = -(-cols // 4) * 4 if aligned else cols + 3
        buf = torch.full((rows, ld), float("nan"), device=DEV)
        buf[:, :cols] = torch.rand((rows, cols), device=DEV, generator=gen).mul_(2).sub_(1)
        return buf[:, :cols]

    A, B, C0 = matrix(M, K), matrix(K, N), torch.rand((M, N), device=DEV, generator=gen)
    for alpha, beta in ((1.0, 0.0), (1.25, -0.5)):
        out = []
        for config in (0, -1):
            C = torch.full((M, N), float("nan"), device=DEV) if beta == 0.0 else C0.clone()
            mfg.gemm(A, B, C, alpha, beta, mode="f32", config=config)
            out.append(C)
        assert torch.isfinite(out[0]).all()
        assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32)), (alpha, beta)


@pytest.mark.parametrize("shape", [(16, 16, 16), (33, 40, 64), (40, 65, 33)], ids=str)
def test_f32_batched_entries_are_bitwise_solo(shape):
    M, N, K = shape
    gen = torch.Generator(device=DEV).manual_seed(M)
    A = torch.rand((29, M, K), device=DEV, generator=gen)
    B = torch.rand((29, K, N), device=DEV, generator=gen)
    C = torch.full((29, M, N), float("nan"), device=DEV)
    mfg.gemm_batched(A, B, C, mode="f32")
    for i in range(29):
        solo = torch.empty((M, N), device=DEV)
        mfg.gemm(A[i], B[i], solo, mode="f32", config=0)
        assert torch.equal(C[i].view(torch.int32), solo.view(torch.int32)), i


F8_SHAPES = [(1, 1, 1), (32, 64, 128), (33, 65, 129), (65, 7, 200), (129, 130, 64), (127, 300, 1003), (777, 610, 330),
             (1100, 1300, 260), (2050, 2300, 515)]


@pytest.mark.parametrize("shape", F8_SHAPES, ids=str)
def test_fp8_default_choice_is_bitwise_the_simple_kernel(shape):
    M, N, K = shape
    gen = torch.Generator(device=DEV).manual_seed(M + 2 * N + K)
    A = torch.rand((M, K), device=DEV, generator=gen).mul_(2).sub_(1)
    B = torch.rand((K, N), device=DEV, generator=gen).mul_(2).sub_(1)
    C0 = torch.rand((M, N), device=DEV, generator=gen)

    def codes(X):  # storage form, rows padded to 16 with NaN codes
        rows, cols = X.shape
        ld = -(-cols // 16) * 16
        buf = torch.full((mfg.convert_bytes(rows, cols, ld, "fp8"),), 0x7F, dtype=torch.uint8, device=DEV)
        mfg.convert(X, buf, ld, "fp8")
        return buf.as_strided((rows, cols), (ld, 1))

    qa, qb = codes(A), codes(B)
    for alpha, beta in ((1.0, 0.0), (1.25, -0.5)):
        out = []
        for config, pre in ((0, True), (-1, True), (0, False), (-1, False)):
            C = torch.full((M, N), float("nan"), device=DEV) if beta == 0.0 else C0.clone()
            mfg.gemm(qa if pre else A, qb if pre else B, C, alpha, beta, mode="fp8", preconverted=pre, config=config)
            out.append(C)
        assert torch.isfinite(out[0]).all()
        for C in out[1:]:
            assert torch.equal(out[0].view(torch.int32), C.view(torch.int32)), (alpha, beta)
