"""FP32 batches on both sides of the rule between the simple and the ring kernel.

Both run the same operations in the same order, so every problem is bitwise
mfg_gemm on that problem alone.
"""
import pytest
import torch

import paper_1803_04014_amd as mfg
from gpu_util import DEV, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("count", [511, 512])
@pytest.mark.parametrize("M,N,K", [(17, 33, 41), (60, 9, 64), (32, 64, 65), (40, 40, 12), (40, 40, 13), (33, 33, 8), (32, 32, 40)])
def test_f32_batch_equals_solo(count, M, N, K):
    gen = torch.Generator(device=DEV).manual_seed(M + 64 * N + 4096 * K)
    A = torch.randn((count, M, K), device=DEV, generator=gen)
    B = torch.randn((count, K, N), device=DEV, generator=gen)
    C = torch.randn((count, M, N), device=DEV, generator=gen)
    C0 = C.clone()
    mfg.gemm_batched(A, B, C, 1.25, -0.5, mode="f32")
    for i in (0, 1, 255, count - 1):
        solo = C0[i].clone()
        mfg.gemm(A[i], B[i], solo, 1.25, -0.5, mode="f32")
        assert torch.equal(C[i].view(torch.int32), solo.view(torch.int32)), i
