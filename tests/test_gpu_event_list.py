"""Event path with the finish-ordered list at the sizes where it changes form:
64 entries in registers and the rest in LDS, the rank bitmap in one register
pair (up to 4096 requests), two (up to 8192) or LDS, its upper level wider than
a wave, finished entries that gather 32 at a time.  Outputs are whole numbers
and equal the oracle's (for the widest bitmap, the ring profile's)."""

import os

import numpy as np
import pytest

import oracle
from paper_2606_22327_amd import svfsim as S
from paper_2606_22327_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("start", "finish", "preempt", "admit_seq")


def run(b, chunks=()):
    with S.Simulator.from_batch(b) as sim:
        for c in chunks:
            sim.step(c)
        sim.run()
        return {p: (sim.read(j), sim.stats(j)) for j, p in enumerate(b.policies)}


def check(b, got):
    for p, (out, st) in got.items():
        r = oracle.run(b, p, threads=min(16, os.cpu_count() or 1))
        for f in FIELDS:
            assert np.array_equal(out[f], r[f]), (b.name, p, f)
        for c, f in enumerate(oracle.STAT_FIELDS):
            if f in st.dtype.names:
                assert np.array_equal(st[f].astype(np.int64), r["stats"][:, c]), (b.name, p, f)


@pytest.mark.parametrize("cap", [1, 63, 64, 65, 128, 0])
def test_list_capacity_around_the_registers(monkeypatch, cap):
    """More requests run at once than the first launch's list holds: it stops
    (also inside a burst) and the continuation resumes it; cap 0: no limit."""
    monkeypatch.setenv("SVFSIM_PROFILE", "list")
    if cap:
        monkeypatch.setenv("SVFSIM_LIST_LDS_CAP", str(cap))
    rng = np.random.default_rng(cap)
    parts = []
    for n, gap in ((0, 0), (1, 0), (64, 0), (65, 0), (200, 0), (333, 1), (500, 3)):
        a = np.cumsum(rng.integers(0, gap + 1, n)) if gap else np.zeros(n, dtype=np.int64)
        parts.append({"arrival": a, "prompt": rng.integers(1, 5, n), "output": rng.integers(1, 150, n)})
    b = W.assemble(f"cap{cap}", parts, 3000, ("svf", "sjf", "fcfs"))
    check(b, run(b))
    check(b, run(b, chunks=(1, 20, 3, 100)))


@pytest.mark.parametrize("n", [63, 64, 65, 4095, 4096, 4097, 8192, 8193])
def test_bitmap_form_boundaries(monkeypatch, n):
    monkeypatch.setenv("SVFSIM_PROFILE", "list")
    rng = np.random.default_rng(n)
    parts = [{"arrival": np.sort(rng.integers(0, n // 2, n)), "prompt": rng.integers(1, 100, n),
              "output": rng.integers(1, 60, n)},
             {"arrival": np.zeros(n, dtype=np.int64), "prompt": rng.integers(1, 100, n),
              "output": rng.integers(1, 20, n)}]
    b = W.assemble(f"n{n}", parts, 4000, ("svf", "fcfs"))
    check(b, run(b))


def test_many_finish_between_two_visits(monkeypatch):
    """200 equal requests finish at one step long before the next arrival: the
    finished entries leave the registers in several rounds."""
    monkeypatch.setenv("SVFSIM_PROFILE", "list")
    parts = []
    for k in (31, 32, 33, 64, 100, 200):
        a = np.concatenate([np.zeros(k), np.full(5, 400), np.full(70, 1000)])
        o = np.concatenate([np.full(k, 5), np.full(5, 300), np.full(70, 7)])
        parts.append({"arrival": a, "prompt": np.full(len(a), 2), "output": o})
    b = W.assemble("together", parts, 2000, ("svf", "sjf", "fcfs"))
    check(b, run(b))
    check(b, run(b, chunks=(3, 3, 500)))


def test_upper_bitmap_level_wider_than_a_wave(monkeypatch):
    """270,000 requests: 66 upper words.  The oracle's scan of the waiting set
    would take hours; the ring profile is the reference."""
    n = 270000
    rng = np.random.default_rng(5)
    part = {"arrival": np.sort(rng.integers(0, 1000, n)), "prompt": rng.integers(1, 64, n),
            "output": rng.integers(1, 32, n)}
    b = W.assemble("wide", [part], 20000, ("svf",))
    got = {}
    for profile in ("ring", "list"):
        monkeypatch.setenv("SVFSIM_PROFILE", profile)
        got[profile] = run(b)["svf"]
    for f in FIELDS:
        assert np.array_equal(got["ring"][0][f], got["list"][0][f]), f
    assert np.array_equal(got["ring"][1], got["list"][1])
    assert (got["list"][1]["status"] == 0).all()
