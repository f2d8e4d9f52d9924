"""mfg_tune_lookup names the configuration a call runs: FP32 operands of the
16-bit kinds are converted into planes with K padded to whole 64-deep stages
from K = 256 on, and the choice is made for that K; a tuned entry counts only
where it serves the shape.  Host code alone: no GPU."""
import numpy as np
import pytest

import paper_1803_04014_amd as mfg
from paper_1803_04014_amd import capi

PRE = capi.MFG_IN_PRECONVERTED


@pytest.fixture(autouse=True)
def _no_table():
    mfg.lib().mfg_tune_clear()
    yield
    mfg.lib().mfg_tune_clear()


@pytest.mark.parametrize("mode", ["f16", "bf16", "refine_a", "split3", "split4", "bf16_split3"])
def test_ragged_k_is_looked_up_as_it_runs(mode):
    look, m = mfg.lib().mfg_tune_lookup, mfg.mode_of(mode)
    g = np.random.default_rng(5)
    shapes = [(1814, 1562, 718), (1410, 1410, 293)] + [tuple(int(v) for v in 2 ** g.uniform(6, 12, 3)) for _ in range(3000)]
    for M, N, K in shapes:
        runs = -(-K // 64) * 64 if K >= 256 else K  # the planes' K, whose choice preconverted planes of that K show
        assert look(M, N, K, m) == look(M, N, runs, m | PRE), (M, N, K)


def test_entries_that_do_not_serve_the_shape(tmp_path):
    look = mfg.lib().mfg_tune_lookup
    shapes = {"fp8": (777, 1234, 1999), "f16": (777, 1234, 1999)}
    default = {m: look(*s, mfg.mode_of(m) | PRE) for m, s in shapes.items()}
    f16 = next(i for i in range(mfg.num_configs("f16")) if mfg.config_name("f16", i).startswith("q256x256"))
    t = tmp_path / "t.txt"
    t.write_text(f"{capi.MFG_FP8_E4M3} 9 10 10 1\n{capi.MFG_F16} 9 10 10 {f16}\n{capi.MFG_F32} 9 10 10 99\n")
    assert mfg.lib().mfg_tune_load(str(t).encode()) == 0
    for m, s in shapes.items():  # K % 128, K % 64 and N % 8 != 0
        assert look(*s, mfg.mode_of(m) | PRE) == default[m]
    assert look(768, 1024, 1024, capi.MFG_FP8_E4M3) == 1 and look(768, 1024, 1024, capi.MFG_F16) == f16
    assert 0 <= look(777, 1234, 1999, capi.MFG_F32) < mfg.num_configs("f32")  # no configuration 99
