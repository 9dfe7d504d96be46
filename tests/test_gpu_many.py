"""ctd_run_many: cases run one after another (their batches sharing launches)
and cases run in rounds over all of them (per-XCD tallies, the event log) leave
the sums of solo runs; a case that may not take all its batches is refused
before any other has run."""
import sys

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


def _read(c):
    s1, hi, lo, nb = c.tally()
    b, st = c.balance(), c.stats()
    assert b.q_incident == b.q_deposited + b.q_escaped
    return s1, hi, lo, nb, b.q_escaped, st.n_steps, st.n_real, st.n_deposits


def _members(ctx, mode, log):
    wls = [W.head(scale=8), W.water_cbct(scale=8), W.tiny()]
    cases = [Case(ctx, wl) for wl in wls]
    for c in cases:
        L.ctd_set_tuning(ctx, c.cs, L.ctd_tuning(256, 5, 16, 1024, mode, 2, 16))
    if log:
        L.ctd_debug_deposit_log(ctx, cases[-1].cs, 0, 1, 64)
    return cases


# none, fewer than the batches, and unequal batches; two calls in a row
@pytest.mark.parametrize("n", [(0, 7, 30_000), (40_003, 0, 1), (20_000, 100_001, 63)])
@pytest.mark.parametrize("mode,log", [(0, False), (1, False), (0, True)])
def test_many_equals_solo(ctx, n, mode, log):
    print(f"[gpu-test] run_many {n} mode {mode} log {log}", flush=True)
    sys.stdout.flush()

    def run(together):
        cases = _members(ctx, mode if together else 0, log and together)
        try:
            for _ in range(2):
                if together:
                    L.ctd_run_many(ctx, [c.cs for c in cases], n)
                else:
                    for c, k in zip(cases, n):
                        c.run(k)
            return [_read(c) for c in cases]
        finally:
            for c in cases:
                c.close()

    for got, ref in zip(run(True), run(False)):
        assert all(np.array_equal(a, b) for a, b in zip(got, ref))


def test_refused_before_any_case_runs(ctx):
    print("[gpu-test] run_many refused by the headroom of its second case", flush=True)
    sys.stdout.flush()
    cases = _members(ctx, 0, False)
    try:
        with pytest.raises(L.CtdError) as e:
            L.ctd_run_many(ctx, [c.cs for c in cases], [1000, 10**12, 1000])
        assert e.value.code == L.CTD_EOVERFLOW
        assert all(c.stats().n_histories == 0 for c in cases)
    finally:
        for c in cases:
            c.close()
