"""The default configuration on both sides of the rules that choose it, between a
kernel without LDS for small problems (configuration 0) and the tiled ones and
among these: shapes timed on an MI355X, the faster one expected.  Host code
alone: no GPU."""
import pytest

import paper_1803_04014_amd as mfg
from paper_1803_04014_amd import capi


@pytest.fixture(autouse=True)
def _no_table():
    mfg.lib().mfg_tune_clear()


def _simple(mode, M, N, K, pre=False):
    return mfg.lib().mfg_tune_lookup(M, N, K, mfg.mode_of(mode) | (capi.MFG_IN_PRECONVERTED if pre else 0)) == 0


# us of a call: configuration 0, the tiled kernel and the transpose it needs
@pytest.mark.parametrize("M,N,K,simple", [
    (64, 64, 64, True),        # 3.8, 6.6
    (896, 128, 64, True),      # 3.8, 6.8
    (64, 192, 64, True),       # 3.8, 6.7
    (3088, 365, 8, True),      # 6.4, 8.8
    (39, 294, 35, True),       # 5.2, 8.7
    (64, 160, 100, True),      # 5.9, 7.5
    (448, 320, 128, True),     # 5.5, 6.7
    (160, 192, 192, True),     # 6.9, 7.4
    (2353, 3090, 22, False),   # 20.3, 14.4
    (5088, 2304, 32, False),   # 22.9, 17.6
    (2336, 5664, 128, False),  # 28.4, 16.5
    (48, 25, 139, False),      # 9.8, 6.8
    (261, 1095, 221, False),   # 13.0, 8.4
    (64, 128, 256, False),     # 8.3, 6.6
    (64, 64, 416, False),      # 13.6, 8.6
])
def test_fp8_codes(M, N, K, simple):
    assert _simple("fp8", M, N, K, pre=True) == simple
    assert not _simple("fp8", M, N, K)  # quantised by the call: B is written transposed


# us of a call: configuration 0, the ring kernel
@pytest.mark.parametrize("M,N,K,simple", [
    (1055, 18, 4, True),      # 2.7, 4.2
    (2641, 56, 5, True),      # 2.7, 4.3
    (96, 2240, 8, True),      # 2.5, 3.6
    (386, 1918, 8, True),     # 3.4, 4.6
    (72, 24, 16, True),       # 2.7, 3.3
    (1825, 1793, 17, True),   # 8.1, 9.4
    (543, 17, 24, True),      # 3.5, 4.2
    (7, 1112, 38, True),      # 4.5, 5.1
    (696, 18, 36, True),      # 4.5, 5.2
    (8, 72, 56, False),       # 4.7, 3.8
    (3241, 2652, 28, False),  # 17.0, 13.6
    (34, 10, 64, False),      # 5.4, 4.8
    (40, 176, 112, False),    # 7.8, 5.3
    (256, 256, 256, False),   # 15, 7.8
    (1000, 1000, 1000, False),
])
def test_f32(M, N, K, simple):
    assert _simple("f32", M, N, K) == simple


# us of a call on preconverted operands: configuration 0, the ring kernel
@pytest.mark.parametrize("mode,M,N,K,simple", [
    ("f16", 136, 232, 8, True),        # 2.6, 3.0
    ("bf16", 480, 32, 16, True),       # 2.3, 3.0
    ("f16", 1936, 704, 16, True),      # 3.5, 4.2
    ("f16", 309, 5, 21, True),         # 2.8, 3.2
    ("f16", 16, 728, 32, True),        # 2.9, 3.1
    ("f16", 8, 112, 40, False),        # 3.2, 2.9
    ("f16", 16, 136, 64, False),       # 3.7, 3.0
    ("f16", 512, 512, 512, False),
    ("refine_a", 1040, 16, 16, True),  # 2.7, 3.5
    ("refine_a", 401, 281, 24, True),  # 3.2, 3.5
    ("split3", 1488, 80, 8, True),     # 3.1, 3.7
    ("split3", 176, 2192, 16, True),   # 3.2, 3.8
    ("split3", 128, 128, 64, False),
    ("bf16_split3", 24, 472, 8, True),
    ("split4", 752, 1248, 16, True),   # 3.6, 4.3
    ("split4", 256, 256, 256, False),
])
def test_16_bit(mode, M, N, K, simple):
    assert _simple(mode, M, N, K, pre=True) == simple


# us of a call on preconverted operands: every configuration of the rule
@pytest.mark.parametrize("mode,M,N,K,config", [
    ("bf16", 1792, 832, 10368, 28),      # 6: 66, 28: 60
    ("f16", 1920, 1024, 6400, 28),       # 6: 46.8, 28: 43.1
    ("f16", 4860, 5751, 716, 29),        # 6: 75.6, 28: 83.7, 30: 79.7, 29: 62.8
    ("f16", 2752, 42432, 128, 29),       # 6: 111, 28: 158, 30: 135, 29: 123
    ("f16", 4374, 12087, 115, 6),        # 6: 51, 28: 71, 30: 68, 29: 63
    ("bf16", 4495, 292, 2982, 6),        # 6: 24, 28: 31
    ("f16", 4096, 4096, 4096, 29),       # 28: 143, 30: 130, 29: 119
    ("refine_a", 4736, 6528, 192, 3),    # 3: 42.8, 7: 52.3, 9: 57.4
    ("refine_a", 1600, 4160, 3008, 7),   # 3: 106, 7: 86, 9: 111
    ("refine_a", 1984, 4992, 1152, 9),   # 3: 59.8, 7: 57.6, 9: 51.5
    ("refine_a", 4941, 2914, 121, 3),    # 3: 19.1, 7: 26.0, 9: 26.3
    ("split3", 4096, 4096, 4096, 9),     # 7: 361, 9: 356
    ("split3", 2048, 4096, 4096, 7),     # 3: 245, 7: 181, 9: 207
    ("split3", 777, 1234, 1999, 3),
    ("split3", 3105, 19080, 118, 3),     # 3: 93, 7: 105, 9: 104
    ("split4", 12480, 832, 448, 2),      # 2: 44.4, 5: 48.9
    ("split4", 9856, 1152, 1152, 5),     # 2: 108, 5: 90
    ("split4", 7468, 4455, 85, 2),       # 2: 58, 5: 71
    ("fp8", 1472, 4096, 2304, 3),        # 256 x 128, 1.16 times what was chosen
])
def test_tiles(mode, M, N, K, config):
    assert mfg.lib().mfg_tune_lookup(M, N, K, mfg.mode_of(mode) | capi.MFG_IN_PRECONVERTED) == config
