"""Preconverted FP8 calls that ask for no storage of the library: a ragged K or
a grid of few tiles is served whatever the size of B, also where the
transposed copy of B that the tiled kernels read cannot be had.  Every result
is bitwise configuration 0's, which reads B's codes as they are."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1803_04014_amd as mfg
from gpu_util import DEV, host, need_gpu

pytestmark = pytest.mark.gpu

MODE = mfg.capi.MFG_FP8_E4M3 | mfg.capi.MFG_IN_PRECONVERTED


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()
    mfg.lib().mfg_tune_clear()


def _codes(rows, cols, seed):
    """A rows x cols matrix in the FP8 storage form (ld rounded up to 16)."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.empty((rows, cols), dtype=torch.float32, device=DEV).uniform_(-1, 1, generator=g)
    ld = -(-cols // 16) * 16
    out = torch.zeros(mfg.convert_bytes(rows, cols, ld, "fp8"), dtype=torch.uint8, device=DEV)
    mfg.convert(x, out, ld, "fp8")
    return out, ld


def _call(fn, M, N, K, a, b, c, *more, stream=None):
    (A, lda), (B, ldb) = a, b
    s = (stream or torch.cuda.current_stream()).cuda_stream
    return getattr(mfg.lib(), fn)(M, N, K, A.data_ptr(), lda, B.data_ptr(), ldb, c.data_ptr(), N, 1.0, 0.0, MODE,
                                  *more, s)


def _both(M, N, K):
    """The operands, an output full of NaN and configuration 0's result."""
    a, b = _codes(M, K, 1), _codes(K, N, 2)
    ref = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    assert _call("mfg_gemm_config", M, N, K, a, b, ref, 0) == 0
    assert bool(torch.isfinite(ref).all())
    return a, b, torch.full_like(ref, float("nan")), ref


# B transposed is 128 MiB against the 64 MiB array (K a multiple of 128, and not)
@pytest.mark.parametrize("M,N,K", [(32, 4096, 32768), (32, 4096, 32700)])
def test_noalloc_beyond_the_array(M, N, K):
    a, b, c, ref = _both(M, N, K)
    assert _call("mfg_gemm_noalloc", M, N, K, a, b, c) == 0
    assert np.array_equal(host(c).view(np.uint32), host(ref).view(np.uint32))


# K / 64 on both sides of the 65535 rows of the transpose's grid
@pytest.mark.parametrize("K", [65535 * 64 - 64, 65536 * 64 + 128, 65536 * 64 + 100])
def test_k_beyond_the_transpose(K):
    a, b, c, ref = _both(16, 16, K)
    assert _call("mfg_gemm", 16, 16, K, a, b, c) == 0
    assert np.array_equal(host(c).view(np.uint32), host(ref).view(np.uint32))


SMALL = [(64, 8192, 8200), (100, 300, 8192)]  # ragged K; K % 128 == 0 on few tiles


@pytest.mark.parametrize("M,N,K", SMALL)
def test_without_memory(M, N, K):
    a, b, c, ref = _both(M, N, K)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert mfg.lib().mfg_fault_inject(0, 1) == 0  # the next allocation fails
    try:
        assert _call("mfg_gemm", M, N, K, a, b, c, stream=st) == 0
    finally:
        mfg.lib().mfg_fault_inject(0, 0)
    assert np.array_equal(host(c).view(np.uint32), host(ref).view(np.uint32))


@pytest.mark.parametrize("M,N,K", SMALL)
def test_captured_and_replayed_past_the_workspace(M, N, K):
    """A captured call holds no memory of the library: replays are right also
    after the capture stream's workspace has been used and has grown."""
    a, b, c, ref = _both(M, N, K)
    st = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        assert _call("mfg_gemm", M, N, K, a, b, c) == 0
    for n in (512, 2048, 4096):  # eager work on that stream, its workspace growing each time
        x = torch.ones((n, n), dtype=torch.float32, device=DEV)
        y = torch.empty_like(x)
        torch.cuda.synchronize()
        mfg.gemm(x, x, y, mode="split3", stream=st.cuda_stream)
        torch.cuda.synchronize()
        c.fill_(float("nan"))
        graph.replay()
        assert np.array_equal(host(c).view(np.uint32), host(ref).view(np.uint32)), n
