"""Per-step path with the running requests in registers, at the sizes where it
changes form: more requests running than the first launch has places for (384),
more evictions at one step than a wave has lanes, entries of the planned
profile with equal finishes removed early, launches that stop inside the
admissions of a step, the bitmap forms, and the limits past which the running
requests stay in memory.  Every output equals the oracle's."""

import os

import numpy as np
import pytest

import oracle
from paper_2606_22327_amd import svfsim as S
from paper_2606_22327_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("start", "finish", "preempt", "admit_seq")


def check(b, chunks=()):
    with S.Simulator.from_batch(b) as sim:
        for c in chunks:
            sim.step(c)
        sim.run()
        got = {p: (sim.read(j), sim.stats(j)) for j, p in enumerate(b.policies)}
    evicted = 0
    for p, (out, st) in got.items():
        r = oracle.run(b, p, threads=min(16, os.cpu_count() or 1))
        for f in FIELDS:
            assert np.array_equal(out[f], r[f]), (b.name, p, f)
        for c, f in enumerate(oracle.STAT_FIELDS):
            if f in st.dtype.names:
                assert np.array_equal(st[f].astype(np.int64), r["stats"][:, c]), (b.name, p, f)
        evicted += int(r["preempt"].sum())
    return evicted


def batch(seed, n, M, s_max, o_max, plan=0, gap=0, instances=4, policies=("svf", "sjf", "fcfs")):
    """plan > 0: one planned length for all; 0: drawn like the true ones."""
    rng = np.random.default_rng(seed)
    parts = []
    for _ in range(instances):
        parts.append({"arrival": np.cumsum(rng.integers(0, gap + 1, n)),
                      "prompt": rng.integers(1, s_max + 1, n), "output": rng.integers(1, o_max + 1, n),
                      "plan_len": np.full(n, plan) if plan else rng.integers(1, o_max + 1, n)})
    return W.assemble(f"step{seed}", parts, M, policies)


@pytest.mark.parametrize("cap", [0, 7, 64, 70])
def test_more_running_than_places(monkeypatch, cap):
    """About 1,000 requests run at once: the first launch stops inside a step
    and the continuation, with room for all, goes on; also with a small list."""
    if cap:
        monkeypatch.setenv("SVFSIM_STEP_LDS_CAP", str(cap))
    check(batch(1, 1200, 5000, 3, 60, gap=1))
    check(batch(2, 1200, 5000, 3, 60, gap=1), chunks=(5, 1, 1, 30, 100))


def test_more_evictions_at_one_step_than_lanes():
    """300 requests planned one step long run on together: the memory grows by
    300 a step and over a hundred leave at once."""
    assert check(batch(3, 300, 1000, 2, 50, plan=1)) > 300
    assert check(batch(4, 300, 1000, 2, 50, plan=1, policies=("svf+cur", "fcfs+cur")),
                 chunks=(1,) * 20) > 300


@pytest.mark.parametrize("plan", [7, 40])
def test_equal_planned_finishes(plan):
    """One planned length: entries of the profile share their finish and leave
    it early or by eviction in any order."""
    check(batch(5, 400, 900, 9, 50, plan=plan))
    check(batch(6, 400, 900, 9, 50, plan=plan, gap=2), chunks=(3, 10, 1, 77))


@pytest.mark.parametrize("n", [64, 65, 4096, 4097, 8192, 8193])
def test_bitmap_form_boundaries(n):
    check(batch(n, n, 20000, 40, 60, gap=2, instances=2, policies=("svf", "svf+cur")))


@pytest.mark.parametrize("limit", ["requests", "budget", "volume", "running"])
def test_limits_of_the_register_form(limit):
    """Both sides of each limit."""
    rng = np.random.default_rng(9)

    def parts(n, s, o):
        return [{"arrival": np.cumsum(rng.integers(0, 8, n)), "prompt": s, "output": o,
                 "plan_len": np.maximum(1, o + rng.integers(-3, 4, n))}]

    if limit == "requests":
        for n in (65536, 65537):
            check(W.assemble(limit, parts(n, rng.integers(1, 30, n), rng.integers(1, 40, n)), 1000,
                             ("fcfs",)))
    elif limit == "budget":
        for M in ((1 << 23) - 2, (1 << 23) - 1):
            check(W.assemble(limit, parts(200, rng.integers(1 << 18, 1 << 20, 200),
                                          rng.integers(4, 60, 200)), M, ("svf", "svf+cur")))
    elif limit == "volume":
        # size and longest plan whose volume is just below 2^31, and just above;
        # the victim is chosen among doubled volumes up to twice that
        s = 20000
        for longest, below in ((48500, True), (48600, False)):
            volume = s * longest + (longest * longest + longest) // 2
            assert (volume < 1 << 31) == below and abs(volume - (1 << 31)) < 1 << 23
            n = 120
            plan = np.where(rng.random(n) < 0.5, longest - rng.integers(0, 3, n),
                            rng.integers(1000, longest, n))
            plan[0] = longest
            part = {"arrival": np.cumsum(rng.integers(0, 2000, n)), "prompt": np.full(n, s),
                    "output": rng.integers(20000, 48000, n), "plan_len": plan}
            assert check(W.assemble(limit, [part] * 2, 1 << 18, ("svf", "fcfs+cur", "svf+cur"))) > 20
    else:
        for n in (2000, 2100):  # all of them fit at once
            check(W.assemble(limit, parts(n, np.full(n, 1), rng.integers(4, 30, n)), 1 << 17, ("svf",)))


@pytest.mark.parametrize("k", [383, 384, 385, 639, 640, 641])
def test_bound_equal_to_the_places(k):
    """Exactly k requests of one token fit at the next step, one more waits:
    with every place taken the launch stops at that candidate, fit or not."""
    n = k + 40
    rng = np.random.default_rng(k)
    o = rng.integers(1, 30, n)
    part = {"arrival": np.zeros(n, dtype=np.int64), "prompt": np.ones(n, dtype=np.int64), "output": o,
            "plan_len": np.maximum(1, o + rng.integers(-2, 3, n))}
    check(W.assemble(f"places{k}", [part] * 3, 2 * k, ("svf+cur", "fcfs+cur", "sjf")))


def one_finish_many_removals(base, per_step, big, M):
    """``base`` small requests run from step 0 to 300, their planned finish too.
    Every step ``per_step`` requests of ``big`` tokens start, planned to finish
    at 300 as well and over after one step: while one entry of the planned
    profile waits for the ``base`` behind it to leave, over 2^31 tokens are
    taken out at 300.  At step 284 one candidate asks for the steps up to 384."""
    rows = [(0, 1, 300, 300)] * base
    for t in range(290):
        if t == 284:
            rows.append((t, 10, 50, 100))
        rows += [(t, big, 1, 300 - t)] * per_step
    a, s, o, plan = (np.array(x, dtype=np.int32) for x in zip(*rows))
    assert base * big > 1 << 31
    return W.assemble(f"one finish {base}", [{"arrival": a, "prompt": s, "output": o, "plan_len": plan}],
                      M, ("fcfs",))


@pytest.mark.parametrize("base,per_step,big", [(560, 2, 4000000), (840, 3, 2600000), (1000, 3, 2600000)])
def test_planned_finish_shared_by_more_than_2_31_tokens_removed(base, per_step, big):
    """In each of the two continuations (in the first launch 384 entries of at most
    M / 2 tokens cannot add up to that)."""
    b = one_finish_many_removals(base, per_step, big, (1 << 23) - 2)
    r = oracle.run(b, "fcfs")
    assert r["start"][base + 284 * per_step] == 284 and int(r["preempt"].sum()) == 0
    check(b)
    check(b, chunks=(100, 150, 20, 10, 5))


@pytest.mark.parametrize("k", [63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("policy", ["fcfs", "svf+cur"])
def test_planned_entries_that_end_in_whole_groups(k, policy):
    """Past the register form's budget the planned profile is read in groups of
    64 from its end: k entries end at step 3, 30 stay, and what they held goes
    to the requests that wait."""
    M, n = (1 << 23) - 1, k + 30
    s = M // (n + 3)
    late = 40
    a = np.concatenate([np.zeros(n), np.ones(late)])
    plan = np.concatenate([np.full(k, 3), np.full(30, 50), np.full(late, 20)])
    o = np.concatenate([np.full(k, 3), np.full(30, 40), np.full(late, 25)])
    part = {"arrival": a, "prompt": np.full(n + late, s), "output": o, "plan_len": plan}
    b = W.assemble(f"groups{k}", [part], M, (policy,))
    r = oracle.run(b, policy)
    assert (r["start"][:n] == 0).all() and (r["start"][n:] == 3).sum() >= 30
    check(b)
    check(b, chunks=(2, 1, 1, 5))
