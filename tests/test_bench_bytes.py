"""The bytes that the benchmark's grouped leg on FP32 operands is priced with:
what the run has to move, not a conversion pass that it may not make."""
import numpy as np

import bench


def test_fp32_grouped_bytes():
    assert bench.fp32_grouped_bytes([(16, 32, 64)]) == 4 * (16 * 64 + 64 * 32 + 16 * 32)
    dims = np.array([[2**20, 2**20, 2**12], [1, 2, 3]], dtype=np.int32)  # past 32 bits
    assert bench.fp32_grouped_bytes(dims) == 4 * (2 * 2**32 + 2**40 + 3 + 6 + 2)
