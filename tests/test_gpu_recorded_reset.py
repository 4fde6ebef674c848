"""A reset recorded into a graph has not run: the next one still clears every
output, and replays of the graph give the same results."""

import numpy as np
import pytest

import oracle
from paper_2606_22327_amd import workloads as W
from paper_2606_22327_amd import svfsim as S

pytestmark = pytest.mark.gpu
KEYS = ("start", "finish", "preempt", "admit_seq")


def test_reset_recorded_but_not_replayed():
    import torch
    b = W.config(2, instances=40)
    ref = oracle.run(b, "svf", threads=8)
    stream = torch.cuda.Stream()
    with S.Simulator.from_batch(b, ("svf",), stream=stream.cuda_stream) as sim:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            sim.reset()
            sim.run()
        sim.reset()                          # the first one that runs
        sim.run()
        got = sim.read(0)
        for k in KEYS:
            assert np.array_equal(got[k], ref[k]), k
        for _ in range(3):
            g.replay()
            sim.run()                        # results change on the device only: read again
            stream.synchronize()
            got = sim.read(0)
            for k in KEYS:
                assert np.array_equal(got[k], ref[k]), k
