"""Reads into host memory: large ones on the per-thread stream (another stream
in each host thread, and large reads use several), and page-locked memory, which
is written directly, beside ordinary memory, which is not."""

import ctypes

import numpy as np
import pytest

import oracle
from paper_2606_22327_amd import svfsim as S
from paper_2606_22327_amd import workloads as W

pytestmark = pytest.mark.gpu
KEYS = ("start", "finish", "preempt", "admit_seq")
PER_THREAD = 2      # hipStreamPerThread


def test_large_read_on_the_per_thread_stream():
    b = W.config(2, instances=600)          # 600,000 requests: 9.6 MB of outputs
    ref = oracle.run(b, "svf", threads=8)
    with S.Simulator.from_batch(b, ("svf",), stream=PER_THREAD) as sim:
        for _ in range(2):
            sim.reset()
            sim.run()
            got = sim.read(0)
            for k in KEYS:
                assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("instances", [4, 600])          # packed and in slots
@pytest.mark.parametrize("locked", [(0, 1, 2, 3), (1, 3), (2,)])
def test_page_locked_destinations(instances, locked):
    import torch
    b = W.config(2, instances=instances)
    ref = oracle.run(b, "svf", threads=8)
    with S.Simulator.from_batch(b, ("svf",)) as sim:
        sim.run()
        bufs = [torch.full((b.num_requests,), -7, dtype=torch.int32, pin_memory=x in locked)
                for x in range(4)]
        rc = S.load().svf_read(sim._h, 0, *(ctypes.c_void_p(t.data_ptr()) for t in bufs), 0)
        assert rc == 0, S.last_error()
        for t, k in zip(bufs, KEYS):
            assert np.array_equal(t.numpy(), ref[k]), k
