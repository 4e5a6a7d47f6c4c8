"""What the batch path's launch settings may and may not slow down.

Times are medians of GPU-event timings of single launches, compared within one
process a few milliseconds apart; each limit stands well between the two cases it
tells apart, whose measured times are given beside it.
"""
import statistics

import numpy as np
import pytest

from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.fixture()
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1812_06545_amd as lib
    lib.ldpc_tuning_clear()
    yield lib
    lib.ldpc_batch_set_threads(512)
    lib.ldpc_tuning_clear()


def _us(call, reps=15):
    import torch
    call()
    times = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    return statistics.median(times)


def test_decode_takes_no_batch_setting(L):
    """ldpc_batch_set_threads is for ldpc_decode_batch: one frame of n = 1944
    through ldpc_decode takes as long under 64 threads as under the default
    (81 us; with the setting applied to it, 473)."""
    import torch
    b = configs.qc1944(2.0, frames=1)
    h = L.Code.from_workload(b.code)
    x = torch.from_numpy(b.llr).cuda()
    ws = torch.empty(L.ldpc_workspace_bytes(h, torch.float32, 1, 10), dtype=torch.uint8, device="cuda")

    def call():
        return L.decode(h, x, 10, workspace=ws)
    usual = _us(call)
    assert L.ldpc_batch_set_threads(64) == 0
    limited = _us(call)
    print(f"[gpu] ldpc_decode {usual:.1f} us, under 64 threads {limited:.1f} us", flush=True)
    assert limited < 2.0 * usual
