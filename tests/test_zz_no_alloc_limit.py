"""svf_run_noalloc at the end of its device scratch: the largest batch that the
documented 128 MiB hold is accepted and right, one request more is refused."""

import numpy as np
import pytest

import oracle
from paper_2606_22327_amd import svfsim as S
from paper_2606_22327_amd import workloads as W

pytestmark = pytest.mark.gpu
LIMIT = 128 << 20
KEYS = ("start", "finish", "preempt", "admit_seq")


def need(sizes, H):
    """Device bytes of a one-policy batch with known lengths and the ring
    profile: each buffer on a 256-byte boundary, 16 bytes of counters last."""
    I, N = len(sizes), int(sum(sizes))
    words = sum((n + 63) // 64 + ((n + 63) // 64 + 63) // 64 for n in sizes)
    parts = [8 * (I + 1), 4, I, 8 * (I + 1), 4 * N, 4 * N, 4 * N, 16 * N, 4 * N, 8 * words,
             4 * I * (H + 64), 4 * N, 80 * I]
    return sum((p + 255) // 256 * 256 for p in parts) + 16


def test_largest_batch_of_the_scratch():
    import torch
    n, H, M = 8000, 8, 1 << 20
    sizes = []
    while need(sizes + [n], H) <= LIMIT:
        sizes.append(n)
    last = next(k for k in range(n, -1, -1) if need(sizes + [k], H) <= LIMIT)
    fits, over = sizes + [last], sizes + [last + 1]
    assert LIMIT - need(fits, H) < 4096 and need(over, H) > LIMIT
    rng = np.random.default_rng(5)
    N = sum(over)
    out = {k: torch.zeros(N, dtype=torch.int32, device="cuda") for k in KEYS}
    stats = torch.zeros(len(over) * S.STATS_DTYPE.itemsize // 8, dtype=torch.int64, device="cuda")
    for sz, good in ((over, False), (fits, True)):
        off = np.zeros(len(sz) + 1, dtype=np.int64)
        off[1:] = np.cumsum(sz)
        a = np.concatenate([np.arange(k, dtype=np.int32) // 4 for k in sz])
        s = rng.integers(1, 9, off[-1]).astype(np.int32)
        o = rng.integers(1, H + 1, off[-1]).astype(np.int32)
        args = (off, a, s, o, M, ("svf",), *(out[k] for k in KEYS), stats)
        if not good:
            with pytest.raises(S.SvfError, match="device scratch"):
                S.run_noalloc(*args, max_steps=1 << 20)
            continue
        S.run_noalloc(*args, max_steps=1 << 20)
        torch.cuda.synchronize()
        b = W.Batch(name="limit", offsets=off, arrival=a, prompt=s, output=o, M=M, policies=("svf",),
                    max_steps=1 << 20)
        ref = oracle.run(b, "svf", threads=8)
        for k in KEYS:
            assert np.array_equal(out[k].cpu().numpy()[:off[-1]], ref[k]), k
