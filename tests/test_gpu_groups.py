"""Batches that share a launch (each with a tally of its own, folded together)
leave the same whole-number sums, counters and maxima as batches run one call
at a time, from one history per batch on, for one case and for several."""
import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W
from tests._helpers import random_phantom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _state(c):
    s1, hi, lo, nb = c.tally()
    b, st = c.balance(), c.stats()
    assert b.q_incident == b.q_deposited + b.q_escaped
    return (s1, hi, lo, nb, b.q_incident, b.q_deposited, b.q_escaped, b.n_histories, st.n_steps,
            st.n_deposits, st.n_escapes, st.n_batches, st.max_s1, st.max_s2_hi)


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def _workload(name):
    if name == "head":
        return W.head(scale=8)            # bound grid, deferred collisions
    if name == "chains":
        wl = W.water_box_bowtie(scale=5)
        wl.geometry["fluence_chains"] = 100
        return wl
    if name == "odd":
        return random_phantom((5, 6, 7), 4, seed=3)
    return W.tiny()


# fewer histories than lanes, than waves; more batches than one launch takes;
# batches with deposit records beside each other
@pytest.mark.parametrize("name,batch,count", [
    ("tiny", 1, 7), ("odd", 65, 130), ("head", 5_000, 10), ("chains", 999, 6),
    ("tiny", 300_000, 3), ("tiny", 40_000_000, 4),
])
def test_grouped_batches_match_single_calls(ctx, name, batch, count):
    print(f"[gpu-test] groups {name} {count} x {batch}", flush=True)
    wl = _workload(name)
    with Case(ctx, wl) as a, Case(ctx, wl) as b:
        L.ctd_run_batches(ctx, a.cs, batch, count)
        for _ in range(count):
            L.ctd_run_batches(ctx, b.cs, batch, 1)
        _same(_state(a), _state(b))
        # the group's tallies were left empty: the next group starts clean
        L.ctd_run_batches(ctx, a.cs, batch, 2)
        L.ctd_run_batches(ctx, b.cs, batch, 1)
        L.ctd_run_batches(ctx, b.cs, batch, 1)
        _same(_state(a), _state(b))


def test_grouped_run_after_a_failure(ctx):
    """A failed group leaves its tallies unfolded; the next group clears them."""
    print("[gpu-test] groups after a failure", flush=True)
    wl = W.tiny(n_histories=50_000)
    with Case(ctx, wl) as a, Case(ctx, wl) as b:
        L.ctd_debug_fail_next_round(ctx)
        with pytest.raises(L.CtdError):
            a.run(wl.n_histories)
        L.ctd_case_reset(ctx, a.cs)
        a.run(wl.n_histories)
        sizes = {wl.n_histories // wl.n_batches}
        assert len(sizes) == 1
        for _ in range(wl.n_batches):
            L.ctd_run_batches(ctx, b.cs, sizes.copy().pop(), 1)
        _same(_state(a), _state(b))


def test_grouped_uneven_cases(ctx):
    """Batched run of cases of different step kinds and uneven, partly empty
    batches against each case alone, batch by batch."""
    print("[gpu-test] groups of uneven cases", flush=True)
    wls = [W.head(scale=8), W.tiny(), random_phantom((4, 4, 9), 3, seed=8)]
    ns = [30_007, 4, 123_456]            # 4 histories in 10 batches: six are empty
    objs = [Case(ctx, wl) for wl in wls]
    try:
        L.ctd_run_many(ctx, [o.cs for o in objs], ns)
        for o, wl, n in zip(objs, wls, ns):
            with Case(ctx, wl) as c:
                for k in range(10):
                    m = n // 10 + (1 if k < n % 10 else 0)
                    if m:
                        L.ctd_run_batches(ctx, c.cs, m, 1)
                _same(_state(o), _state(c))
    finally:
        for o in objs:
            o.close()
