"""Large reads on the per-thread stream: another stream in each host thread,
and large reads use several."""

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
