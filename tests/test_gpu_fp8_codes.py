"""FP8 codes at every rounding boundary, with and without a NaN in the tile.

The codes come from the hardware conversion except in wavefronts that hold a
NaN or an infinity: both ways give the oracle's codes for every finite value,
and a NaN keeps its sign.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1803_04014_amd as mfg
from gpu_util import DEV, dev, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def boundaries():
    """Every E4M3 value, the midpoints between neighbours and their FP32 neighbours, both signs, and tiny values."""
    code = np.arange(127)
    e, f = code >> 3, code & 7
    val = np.where(e == 0, f * 2.0 ** -9, (1 + f / 8) * 2.0 ** (e - 7.0)).astype(np.float32)
    mid = ((val[1:] + val[:-1]) / 2).astype(np.float32)
    pts = np.concatenate([val, mid, np.nextafter(mid, np.float32(np.inf)), np.nextafter(mid, np.float32(0)),
                          np.float32([2.0 ** -149, 2.0 ** -126, 2.0 ** -60])])
    return np.concatenate([pts, -pts])


def quantize(X):
    codes = torch.empty(X.shape, dtype=torch.uint8, device=DEV)
    scales = torch.empty((-(-X.shape[0] // 128), -(-X.shape[1] // 128)), dtype=torch.float32, device=DEV)
    mfg.quantize_fp8(dev(X), codes, scales)
    return host(codes), host(scales)


@pytest.mark.parametrize("exponent", [0, -100, 90])
@pytest.mark.parametrize("shape", [(128, 128), (200, 150)])
def test_codes_at_boundaries(shape, exponent):
    pts = boundaries()
    X = (np.resize(pts, shape) * np.float32(2.0 ** exponent)).astype(np.float32)
    X[::128, ::128] = np.float32(448.0 * 2.0 ** exponent)  # every tile's scale is 2^exponent
    codes, scales = quantize(X)
    q = oracle.fp8_quantize(X)
    assert np.array_equal(scales, np.full_like(scales, 2.0 ** exponent))
    assert np.array_equal(codes, q.codes)
    Y = X.copy()
    Y[3, 5], Y[70, 90] = np.nan, -np.float32(np.nan)
    got, _ = quantize(Y)
    special = np.isnan(Y)
    assert np.array_equal(got[~special], codes[~special])
    assert got[3, 5] & 0x7F == 0x7F and got[70, 90] & 0x7F == 0x7F
    assert [bool(got[3, 5] & 0x80), bool(got[70, 90] & 0x80)] == [bool(np.signbit(Y[3, 5])), bool(np.signbit(Y[70, 90]))]
