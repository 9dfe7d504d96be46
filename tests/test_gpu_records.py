"""Deposit records: launches that append their deposits to per-bucket chains
which a second kernel sums must leave the same whole-number tallies as the
launches that add every deposit to the tally (the event-log launches and the
launches below the size limits do), at the edges of buckets and segments."""
import sys
from dataclasses import replace

import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
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


def _sums(ctx, wl, batch, count, log):
    with Case(ctx, wl) as c:
        if log:   # a launch with the event log adds every deposit to the tally
            L.ctd_debug_deposit_log(ctx, c.cs, 0, 1, 64)
        L.ctd_run_batches(ctx, c.cs, batch, count)
        s1, hi, lo, nb = c.tally()
        b, st = c.balance(), c.stats()
        assert b.q_incident == b.q_deposited + b.q_escaped
        assert int(s1.sum()) == b.q_deposited
        return s1, hi, lo, nb, b.q_deposited, st.n_deposits


# one voxel; fewer voxels than buckets; a last bucket of one voxel; buckets of
# 2^k voxels with a remainder; all deposits in few buckets (pencil), in all
# (cone); histories from the smallest launch that keeps records on
@pytest.mark.parametrize("shape,pencil,batch", [
    ((1, 1, 1), True, 200_000), ((3, 3, 3), True, 200_001), ((5, 13, 1), False, 250_000),
    ((32, 32, 32), True, 400_000), ((33, 31, 37), False, 1_000_003),
    ((16, 16, 16), True, 6_000_000), ((97, 61, 50), False, 2_000_000),
])
def test_records_match_the_tally(ctx, shape, pencil, batch):
    print(f"[gpu-test] records {shape} pencil={pencil} {batch}", flush=True)
    sys.stdout.flush()
    wl = _box(*shape, pencil)
    a, b = _sums(ctx, wl, batch, 2, False), _sums(ctx, wl, batch, 2, True)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    assert int(a[0].sum()) > 0


def test_records_of_uneven_cases(ctx):
    """Workgroups that change case close their chains: a batched run of three
    record-keeping cases equals the cases alone."""
    print("[gpu-test] records of a batched run", flush=True)
    wls = [_box(8, 8, 8, True), _box(40, 30, 20, False), _box(32, 32, 32, True)]
    ns = [3_000_000, 700_000, 1_500_001]
    objs = [Case(ctx, wl) for wl in wls]
    try:
        L.ctd_run_many(ctx, [o.cs for o in objs], ns)
        for o, wl, n in zip(objs, wls, ns):
            s1, hi, lo, nb = o.tally()
            with Case(ctx, wl) as c:
                L.ctd_debug_deposit_log(ctx, c.cs, 0, 1, 64)
                c.run(n)
                r1, rhi, rlo, rnb = c.tally()
            assert nb == rnb and np.array_equal(s1, r1)
            assert np.array_equal(hi, rhi) and np.array_equal(lo, rlo)
    finally:
        for o in objs:
            o.close()
