"""Validation on several host threads (batches of 2^20 requests and more): the
first error in instance order is the one reported, as on one thread.  Needs no
GPU: malformed batches are refused before any device call."""

import numpy as np
import pytest

from paper_2606_22327_amd import svfsim as S

I, N = 40, 30000   # 1.2 million requests


def batch():
    return dict(offsets=np.arange(I + 1, dtype=np.int64) * N,
                arrival=np.tile(np.arange(N, dtype=np.int32), I),
                prompt=np.full(I * N, 3, dtype=np.int32), output=np.full(I * N, 5, dtype=np.int32))


@pytest.mark.parametrize("where", [(0, 0), (0, N - 1), (19, 7), (20, 0), (I - 1, N - 1)])
@pytest.mark.parametrize("what,text,code", [
    ("arrival", "arrivals not in order", -1), ("prompt", "prompt -2147483648 < 1", -1),
    ("output", "output 0 < 1", -1), ("large", "exceeds M", -4)])
def test_first_error_in_instance_order(where, what, text, code):
    b = batch()
    for i, j in (where, (min(where[0] + 5, I - 1), N - 1)):   # a later one too
        k = i * N + j
        if what == "arrival":
            if j == 0:
                continue          # the first request of an instance follows nothing
            b["arrival"][k] = 0 if j > 0 else 1
        elif what == "prompt":
            b["prompt"][k] = -2 ** 31
        elif what == "output":
            b["output"][k] = 0
        else:
            b["output"][k] = 2 ** 31 - 1
    if what == "arrival" and where[1] == 0:
        where = (min(where[0] + 5, I - 1), N - 1)
    with pytest.raises(S.SvfError) as e:
        S.Simulator(b["offsets"], b["arrival"], b["prompt"], b["output"], 1000, ("svf", "fcfs"),
                    max_steps=10)
    assert e.value.code == code
    assert text in str(e.value) and f"instance {where[0]}" in str(e.value)
    assert f"request {where[1]}" in str(e.value)
