"""The tuner on shapes whose default choice is no explicit configuration (a
ragged K, rows that are not 16-byte aligned): it times the default too, so a
call on the tuned shape runs what it ran before, or something faster."""
import numpy as np
import pytest
import torch

import paper_1803_04014_amd as mfg
from gpu_util import DEV, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()
    mfg.lib().mfg_tune_clear()
    yield
    mfg.lib().mfg_tune_clear()


def _served(mode, M, N, K, pre, index):
    """Whether `index` serves the operands as an explicit configuration."""
    a, b, c = _operands(mode, M, N, K, pre)
    try:
        mfg.gemm(a, b, c, mode=mode, preconverted=pre, config=index)
        return True
    except mfg.MfgError as e:
        assert e.status == mfg.capi.MFG_ERR_UNSUPPORTED
        return False


def _operands(mode, M, N, K, pre):
    g = torch.Generator(device=DEV).manual_seed(7)

    def rand(rows, cols):  # preconverted: whole 16-byte pieces; FP32: contiguous rows of any alignment
        ld = -(-cols // 8) * 8 if pre else cols
        x = torch.empty((rows, ld), dtype=torch.float32, device=DEV).uniform_(-1, 1, generator=g)
        return (x.half() if pre else x)[:, :cols]

    return rand(M, K), rand(K, N), torch.zeros((M, N), dtype=torch.float32, device=DEV)


# the simple kernel takes 2 to 11 times as long as the default on each of these
@pytest.mark.parametrize("mode,M,N,K,pre", [
    ("fp8", 777, 1234, 1999, False),   # K % 128 != 0: only the simple kernel is explicit
    ("f32", 1772, 2735, 1437, False),  # odd ld: likewise
])
def test_default_is_kept_where_it_is_fastest(mode, M, N, K, pre):
    m = mfg.mode_of(mode)
    default = mfg.lib().mfg_tune_lookup(M, N, K, m)
    assert default > 0 and not _served(mode, M, N, K, pre, default)
    a, b, c = _operands(mode, M, N, K, pre)
    want = torch.empty_like(c)
    mfg.gemm(a, b, want, mode=mode, preconverted=pre)
    best, ms = mfg.autotune(a, b, c, mode, reps=3, preconverted=pre)
    assert best == default and ms > 0
    assert mfg.lib().mfg_tune_lookup(M, N, K, m) == default
    mfg.gemm(a, b, c, mode=mode, preconverted=pre)
    assert np.array_equal(host(c).view(np.uint32), host(want).view(np.uint32))


@pytest.mark.parametrize("mode,M,N,K", [("f16", 4000, 4000, 4001), ("bf16", 1030, 1036, 1100), ("fp8", 100, 130, 300)])
def test_tuned_call_takes_no_longer(mode, M, N, K):
    pre = mode != "fp8"
    a, b, c = _operands(mode, M, N, K, pre)
    if mode == "bf16":
        a, b = a.to(torch.bfloat16), b.to(torch.bfloat16)

    def us():
        t = []
        for _ in range(9):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            for _ in range(20):
                mfg.gemm(a, b, c, mode=mode, preconverted=pre)
            e.record()
            torch.cuda.synchronize()
            t.append(s.elapsed_time(e) * 50)
        return min(t)

    us()
    before = us()
    mfg.autotune(a, b, c, mode, reps=5, preconverted=pre)
    after = us()
    assert after <= 1.15 * before, (before, after)
