"""What the server's slots hold for converted operands stays within the budget,
idle slots included: by the scheduler's own count (MFG_LOG lines) in a dry run
and on the GPU, and by the device's free memory."""
import os
import re
import subprocess
import sys
import threading

import pytest
import torch

import paper_1803_04014_amd as mfg
from gpu_util import DEV, need_gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# Small groups on every slot, requests of the slots' share and of the whole
# budget among them, so that arenas grow, are given up and are replaced.
TRACE = """
import sys, numpy as np, paper_1803_04014_amd as mfg
dev, budget, slots = int(sys.argv[1]), int(sys.argv[2]), int(sys.argv[3])
g = np.random.default_rng(3)
ptr = dict(A_ptr=0x7F0000000000, B_ptr=0x7F1000000000, C_ptr=0x7F2000000000)
if dev >= 0:
    import torch
    buf = [torch.ones(1 << 22, dtype=torch.float32, device="cuda:0") for _ in range(3)]
    ptr = dict(zip(ptr, (b.data_ptr() for b in buf)))
    torch.cuda.synchronize()
s = mfg.Server(budget, slots=slots, device=dev, max_group=4)
t = []
for i in range(160):
    n = int(2 ** g.uniform(5, 10)) if i % 8 else 1440   # split3 of 1440: 2 * 8 MiB, the budget nearly whole
    mode = ["split3", "f16", "fp8", "f32"][i % 4] if i % 8 else "split3"
    t.append(s.submit(None, None, None, mode, M=n, N=n, K=n, lda=n, ldb=n, ldc=n, **ptr))
    if i % 40 == 39:
        s.drain()
s.drain()
st = s.stats()
assert st["completed"] == 160 and st["failed"] == 0 and st["bytes_in_use"] == 0, st
s.close()
"""


def _held(device, budget, slots):
    env = dict(os.environ, MFG_LOG="1", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", TRACE, str(device), str(budget), str(slots)], capture_output=True,
                       text=True, env=env, cwd=ROOT, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return [int(x) for x in re.findall(r"mfg_server: .* held (\d+)", r.stderr)]


@pytest.mark.parametrize("slots", [1, 4])
def test_slots_hold_at_most_the_budget_dry(slots):
    budget = 17 << 20
    held = _held(-1, budget, slots)
    assert len(held) > 40 and max(held) <= budget
    assert max(held) > budget // 2  # the large requests were held


@pytest.mark.gpu
@pytest.mark.parametrize("slots", [1, 4])
def test_slots_hold_at_most_the_budget(slots):
    need_gpu()
    budget = 17 << 20
    held = _held(0, budget, slots)
    assert len(held) > 40 and max(held) <= budget


@pytest.mark.gpu
def test_device_memory_of_a_large_request_beside_grown_slots():
    need_gpu()
    budget, n = 512 << 20, 4096  # split3 of 4096: 128 MiB of planes; of 8192: the whole budget
    big = [torch.ones((8192, 8192), dtype=torch.float32, device=DEV) for _ in range(3)]
    part = [[x[:n, :n] for x in big[:2]] + [torch.empty((n, n), dtype=torch.float32, device=DEV)] for _ in range(4)]
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    s = mfg.Server(budget, slots=4, max_group=1)
    staged = free0 - torch.cuda.mem_get_info()[0]
    for _ in range(6):  # every slot's storage grows
        for a, b, c in part:
            s.submit(a, b, c, "split3")
        s.drain()
    least, done = [free0], threading.Event()

    def watch():
        while not done.is_set():
            least[0] = min(least[0], torch.cuda.mem_get_info()[0])

    w = threading.Thread(target=watch)
    w.start()
    for _ in range(5):
        s.submit(big[0], big[1], big[2], "split4")
        s.drain()
    done.set()
    w.join()
    stats = s.stats()
    s.close()
    assert stats["failed"] == 0 and stats["completed"] == 29
    # (the runtime rounds allocations, and loads kernels on their first use)
    assert free0 - staged - least[0] <= budget + (96 << 20)


@pytest.mark.gpu
def test_growing_storage_does_not_wait_for_other_slots():
    """Requests whose slot needs more storage each time finish beside a long
    request on the other slot."""
    need_gpu()
    n = 16384
    x, y = (torch.ones((n, n), dtype=torch.float32, device=DEV) for _ in range(2))
    c = torch.empty_like(x)
    # 520 x 520 x K in F16: 8, 40 and 120 MiB of planes, and tiles that find room
    # beside the long request's
    small = [tuple(torch.ones(d, dtype=torch.float32, device=DEV) for d in ((520, k), (k, 520), (520, 520)))
             for k in (4096, 20480, 61440)]
    s = mfg.Server(4 << 30, slots=2, max_group=1)
    s.submit(*small[0], "f16")  # (kernels loaded, the first allocation made)
    s.drain()
    torch.cuda.synchronize()
    long = s.submit(x, y, c, "f32")  # about 70 ms
    ends = []
    for a, b, out in small:
        t = s.submit(a, b, out, "f16")
        while True:
            st, r = s.poll(t)
            if st != mfg.capi.MFG_PENDING:
                break
        assert st == 0
        ends.append(r["t_end_ns"])
    s.drain()
    st, r = s.poll(long)
    s.close()
    assert st == 0 and max(ends) < r["t_end_ns"]
