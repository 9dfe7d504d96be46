"""What launches do at their limits: deposit records whose segments run out
part-way (the rest goes to the tally), and launches of several cases (run in
rounds) with records of different bucket sizes and with different kinds of step.
Sums are whole numbers and equal those of the launches without limits."""
import sys
from dataclasses import replace

import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W
from tests._helpers import random_phantom

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _box(nx, ny, nz, pencil):
    """A water box of the given voxel counts, 16 x 16 x 16 cm."""
    base = W.tiny() if pencil else W.water_box_bowtie(scale=5)
    g = dict(nx=nx, ny=ny, nz=nz, dx=16.0 / nx, dy=16.0 / ny, dz=16.0 / nz, ox=-8.0, oy=-8.0,
             oz=-8.0)
    geo = dict(base.geometry)
    if pencil:
        geo["src"] = (0.01, 0.02, -8.0)
    return replace(base, grid=g, geometry=geo, mat=np.zeros((nz, ny, nx), np.uint8),
                   rho=np.ones((nz, ny, nx), np.float32))


def _state(c):
    s1, hi, lo, nb = c.tally()
    b, st = c.balance(), c.stats()
    assert b.q_incident == b.q_deposited + b.q_escaped
    assert int(s1.sum()) == b.q_deposited
    return (s1, hi, lo, nb, b.q_deposited, b.q_escaped, st.n_steps, st.n_deposits, st.max_s1,
            st.max_s2_hi)


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


# fewer segments than buckets, one per bucket and some, enough for a part of
# the histories; one voxel (one bucket takes every deposit)
@pytest.mark.parametrize("segments", [1, 70, 200])
@pytest.mark.parametrize("shape,pencil,batch", [
    ((1, 1, 1), True, 20_000_000), ((32, 32, 32), True, 20_000_000),
    ((33, 31, 37), False, 10_000_003),
])
def test_records_run_out(ctx, shape, pencil, batch, segments):
    print(f"[gpu-test] {segments} segments {shape} pencil={pencil} {batch}", flush=True)
    sys.stdout.flush()
    wl = _box(*shape, pencil)
    with Case(ctx, wl) as a, Case(ctx, wl) as b:
        L.ctd_debug_limits(ctx, record_segments=segments)
        L.ctd_run_batches(ctx, a.cs, batch, 2)
        launches, records = L.ctd_debug_launches(ctx)
        assert records == launches > 0
        grid = 256 * 5     # workgroups of the default launch on 256 CUs
        if segments <= 70:   # more deposits than the launches' segments hold
            assert a.stats().n_deposits > launches * grid * segments * 256
        L.ctd_debug_limits(ctx)
        L.ctd_debug_deposit_log(ctx, b.cs, 0, 1, 64)   # adds every deposit to the tally
        L.ctd_run_batches(ctx, b.cs, batch, 2)
        assert L.ctd_debug_launches(ctx)[1] == records
        _same(_state(a), _state(b))


def test_too_little_memory_for_records(ctx):
    """A launch whose records would find less than 1/32 of the room it wants
    (1.2 GB here) adds its deposits to the tally; with more it keeps what it
    can, also in a block made for another launch."""
    print("[gpu-test] records by memory", flush=True)
    wl = _box(32, 32, 32, False)
    with Case(ctx, wl) as a, Case(ctx, wl) as b:
        L.ctd_debug_deposit_log(ctx, b.cs, 0, 1, 64)
        for free, batch, recorded in [(200, 30, 0), (600, 30, 1), (0, 1, 1), (1, 30, 1)]:
            n0, r0 = L.ctd_debug_launches(ctx)
            # MB; an eighth of what is free counts
            L.ctd_debug_limits(ctx, memory_bytes=free * 1_000_000)
            L.ctd_run_batches(ctx, a.cs, batch * 1_000_000, 1)
            n1, r1 = L.ctd_debug_launches(ctx)
            assert (n1 - n0, r1 - r0) == (1, recorded)
            L.ctd_debug_limits(ctx)
            L.ctd_run_batches(ctx, b.cs, batch * 1_000_000, 1)
            _same(_state(a), _state(b))


@pytest.mark.parametrize("segments", [0, 20])
def test_records_of_several_cases_in_a_launch(ctx, segments):
    print(f"[gpu-test] records in rounds, {segments} segments", flush=True)
    wls = [_box(8, 8, 8, True), _box(40, 30, 20, False), _box(97, 61, 50, False),
           _box(32, 32, 32, True), _box(1, 1, 1, True)]
    ns = [3_000_000, 700_000, 2_000_003, 1_500_001, 40_000]
    objs = [Case(ctx, wl) for wl in wls]
    try:
        L.ctd_debug_limits(ctx, record_segments=segments, rounds=True)
        L.ctd_run_many(ctx, [o.cs for o in objs], ns)
        launches, records = L.ctd_debug_launches(ctx)
        assert (launches, records) == (1, 1)
        L.ctd_debug_limits(ctx)
        for o, wl, n in zip(objs, wls, ns):
            with Case(ctx, wl) as c:
                L.ctd_debug_deposit_log(ctx, c.cs, 0, 1, 64)
                c.run(n)
                _same(_state(o), _state(c))
    finally:
        for o in objs:
            o.close()


def test_kinds_of_step_in_shared_rounds(ctx):
    """Batches of several cases share launches, one per kind of step; some
    batches are empty."""
    print("[gpu-test] kinds of step in shared rounds", flush=True)
    wls = [W.head(scale=8), W.tiny(), random_phantom((4, 4, 9), 3, seed=8)]
    ns = [30_007, 4, 123_456]            # 4 histories in 10 batches: six are empty
    objs = [Case(ctx, wl, tracking=L.CTD_TRACK_MACRO if i == 2 else None)
            for i, wl in enumerate(wls)]
    try:
        L.ctd_debug_limits(ctx, rounds=True)
        L.ctd_run_many(ctx, [o.cs for o in objs], ns)
        assert L.ctd_debug_launches(ctx)[0] == 3
        for o, wl, n, i in zip(objs, wls, ns, range(3)):
            with Case(ctx, wl, tracking=L.CTD_TRACK_MACRO if i == 2 else None) as c:
                for k in range(10):
                    m = n // 10 + (1 if k < n % 10 else 0)
                    if m:
                        L.ctd_run_batches(ctx, c.cs, m, 1)
                _same(_state(o), _state(c))
    finally:
        for o in objs:
            o.close()
