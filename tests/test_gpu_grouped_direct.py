"""Grouped plans whose kernel converts FP32 operands itself.

Every problem is held bitwise to mfg_gemm on its FP32 operands alone.  Sizes
sit at the edges of tiles, blocks and 4-element loads; rows start at any
element; NaN surrounds every operand, so a value read beyond its row or its
last row would show.  Plans past the direct path's largest side, or with a C
that overlaps an operand, read every operand before any C is written.
"""
import pytest
import torch

import paper_1803_04014_amd as mfg
from gpu_util import DEV, need_gpu

pytestmark = pytest.mark.gpu

MODES = ["f16", "bf16", "refine_a", "split3", "split4", "bf16_split3"]
DIMS = [(1, 1, 1), (2, 3, 5), (63, 64, 65), (64, 65, 63), (65, 63, 64), (128, 128, 128), (129, 127, 193), (7, 300, 1), (300, 6, 2),
        (33, 131, 66), (1, 768, 130), (768, 2, 67), (256, 255, 254), (5, 9, 0), (0, 4, 4)]


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def operand(rows, cols, ld, offset, gen):
    buf = torch.full((offset + rows * ld + 64,), float("nan"), device=DEV)
    view = buf.as_strided((rows, cols), (ld, 1), offset)
    view.copy_(torch.randn((rows, cols), device=DEV, generator=gen))
    return view


def check(problems, mode):
    """The plan's results against each problem alone, on copies taken before the run."""
    alone = []
    for A, B, C in problems:
        out = C.clone()
        mfg.gemm(A.clone(), B.clone(), out, 0.75, 0.5, mode=mode)
        alone.append(out)
    plan = mfg.GroupedPlan(problems, mode, fp32_in=True)
    plan.run(0.75, 0.5)
    torch.cuda.synchronize()
    plan.close()
    for i, ((A, B, C), out) in enumerate(zip(problems, alone)):
        assert torch.equal(C.contiguous().view(torch.int32), out.contiguous().view(torch.int32)), (mode, i, A.shape, B.shape)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("largest", [768, 769])
def test_direct_equals_solo(mode, largest):
    gen = torch.Generator(device=DEV).manual_seed(largest)
    problems = []
    for i, (M, N, K) in enumerate(DIMS + [(largest, 40, 70)]):
        pad, off = i % 5, i % 3
        problems.append((operand(M, K, max(1, K) + pad, off, gen), operand(K, N, N + (i % 4), (i + 1) % 4, gen),
                         torch.randn((M, N), device=DEV, generator=gen)))
    check(problems, mode)


@pytest.mark.parametrize("mode", ["f16", "split3"])
def test_output_overlapping_an_operand(mode):
    gen = torch.Generator(device=DEV).manual_seed(3)
    n, buf = 96, torch.empty((97, 96), device=DEV)
    buf.copy_(torch.randn((97, 96), device=DEV, generator=gen))
    other = [torch.randn((n, n), device=DEV, generator=gen) for _ in range(60)]
    chained = [(other[i], other[i + 1], other[i + 2]) for i in range(0, 57, 3)]
    shared = (buf[1:], other[57], other[58])  # its A shares rows with the next problem's C
    check(chained + [shared, (other[59], other[0], buf[:96])], mode)


# us with the pass, and converted in the kernel
@pytest.mark.parametrize("mode,count,M,N,K,in_kernel", [
    ("f16", 4, 128, 128, 32768, False),   # 517, 761
    ("f16", 64, 512, 512, 512, True),     # 68, 49
    ("f16", 16, 768, 768, 512, True),     # 39, 36
    ("bf16", 2, 256, 256, 8192, False),   # 130 to 141, 188 to 191
    ("split3", 64, 128, 128, 2048, True),  # 75, 41
    ("refine_a", 16, 768, 768, 8192, False),  # 810, 899
    ("refine_a", 4, 768, 768, 512, True),  # 23, 19
])
def test_conversion_where_it_costs_less(mode, count, M, N, K, in_kernel):
    """Only a plan with a pass holds converted copies: 16 MB of them here at least."""
    gen = torch.Generator(device=DEV).manual_seed(K)
    problems = [(torch.randn((M, K), device=DEV, generator=gen), torch.randn((K, N), device=DEV, generator=gen),
                 torch.randn((M, N), device=DEV, generator=gen)) for _ in range(count)]
    check(problems[:2], mode)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plan = mfg.GroupedPlan(problems, mode, fp32_in=True)
    held = before - torch.cuda.mem_get_info()[0]
    plan.close()
    copies = 2 * count * K * (M + N)
    assert held < copies / 2 if in_kernel else held >= copies / 2, held
