"""Alg. A1 beamlets of batches that share a launch: a case's own buffer holds
one batch and stays where it is (ctd_run_batches_static enqueues its address),
and where the memory allows no more, the batches run one at a time."""
import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _chains(n):
    wl = W.water_box_bowtie(scale=5)
    wl.geometry["fluence_chains"] = n
    return wl


def _group_tallies(ctx, batches):
    """Let the context make the tallies of a launch of so many batches, by a
    case of the same grid without chains; the bytes they take."""
    wl = W.water_box_bowtie(scale=5)
    with Case(ctx, wl) as c:
        L.ctd_run_batches(ctx, c.cs, 100, batches)
        return 8 * c.V * (batches - 1)


def _state(c):
    s1, hi, lo, nb = c.tally()
    b, st = c.balance(), c.stats()
    assert b.q_incident == b.q_deposited + b.q_escaped
    return s1, hi, lo, nb, b.q_deposited, st.n_steps, st.n_deposits


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("batch", [1, 999, 200_000])
def test_no_room_for_the_beamlets_of_a_group(ctx, batch):
    print(f"[gpu-test] beamlets of one batch of {batch} only", flush=True)
    wl, count = _chains(100), 7
    with Case(ctx, wl) as a, Case(ctx, wl) as b:
        held = _group_tallies(ctx, count)
        n0 = L.ctd_debug_launches(ctx)[0]
        # the batch's beamlets, no more
        L.ctd_debug_limits(ctx, memory_bytes=held + 4 * batch + 3)
        L.ctd_run_batches(ctx, a.cs, batch, count)
        assert L.ctd_debug_launches(ctx)[0] - n0 == count
        L.ctd_debug_limits(ctx)
        for _ in range(count):
            L.ctd_run_batches(ctx, b.cs, batch, 1)
        _same(_state(a), _state(b))


@pytest.mark.parametrize("chains", [1, 100])
def test_own_buffer_stays(ctx, chains):
    """After a batch has sized it, runs of more batches of that size, grouped
    and through the static entry point, allocate nothing for the case."""
    print(f"[gpu-test] beamlet buffer stays, {chains} chains", flush=True)
    wl, batch = _chains(chains), 20_000
    with Case(ctx, wl) as a, Case(ctx, wl) as b:
        _group_tallies(ctx, 3)
        L.ctd_run_batches(ctx, a.cs, batch, 1)
        L.ctd_debug_limits(ctx, memory_bytes=1)
        L.ctd_run_batches(ctx, a.cs, batch, 3)
        L.ctd_debug_limits(ctx)
        n0 = L.ctd_debug_launches(ctx)[0]
        L.ctd_run_batches(ctx, a.cs, batch, 4)
        assert L.ctd_debug_launches(ctx)[0] - n0 == 1
        L.ctd_run_batches_static(ctx, a.cs, batch, 2)
        for _ in range(10):
            L.ctd_run_batches(ctx, b.cs, batch, 1)
        _same(_state(a), _state(b))


def test_static_entry_after_a_grouped_run(ctx):
    """A grouped run sizes the buffer for one batch, and not for all."""
    print("[gpu-test] static entry after a grouped run", flush=True)
    with Case(ctx, _chains(100)) as c:
        L.ctd_run_batches(ctx, c.cs, 5_000, 6)
        L.ctd_run_batches_static(ctx, c.cs, 5_000, 1)
        with pytest.raises(L.CtdError) as e:
            L.ctd_run_batches_static(ctx, c.cs, 5_001, 1)
        assert e.value.code == L.CTD_EINVAL


def test_run_many_refused_for_a_later_case(ctx):
    """A batched run whose last case cannot have its beamlets leaves every case
    as it was; with the memory it equals the cases alone."""
    print("[gpu-test] run_many without memory for its last case", flush=True)
    wls = [W.tiny(), W.head(scale=8), _chains(100)]
    ns = [20_000, 10_001, 30_000_000]
    objs = [Case(ctx, wl) for wl in wls]
    try:
        for rounds in (False, True):
            L.ctd_debug_limits(ctx, memory_bytes=4_000_000, rounds=rounds)
            with pytest.raises(L.CtdError) as e:
                L.ctd_run_many(ctx, [o.cs for o in objs], ns)
            assert e.value.code == L.CTD_ENOMEM
            assert all(o.stats().n_histories == 0 and o.stats().n_batches == 0 for o in objs)
        L.ctd_debug_limits(ctx)
        L.ctd_run_many(ctx, [o.cs for o in objs], ns)
        for o, wl, n in zip(objs, wls, ns):
            with Case(ctx, wl) as c:
                c.run(n)
                _same(_state(o), _state(c))
    finally:
        for o in objs:
            o.close()
