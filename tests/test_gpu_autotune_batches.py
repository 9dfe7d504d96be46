"""ctd_autotune keeps a configuration that is fast for several batches of the
trial's size, which share launches under tally mode 0, and not only for one;
the case's own histories are left alone."""
import time

import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W

pytestmark = pytest.mark.gpu


def test_kept_configuration_runs_batches_as_fast_as_the_default():
    print("[gpu-test] autotune over batches", flush=True)
    batch, count = 1_000_000, 10
    ctx = L.ctd_create(0)
    try:
        with Case(ctx, W.water_cbct(scale=8)) as c:
            default = L.ctd_get_tuning(ctx, c.cs)
            L.ctd_run_batches(ctx, c.cs, batch, 2)
            before = c.tally()
            best = L.ctd_autotune(ctx, c.cs, batch)
            for x, y in zip(c.tally(), before):
                assert np.array_equal(x, y)
            took = {}
            for _ in range(9):               # in turn: the fastest of each
                for name, t in (("default", default), ("kept", best)):
                    L.ctd_set_tuning(ctx, c.cs, t)
                    L.ctd_case_reset(ctx, c.cs)
                    t0 = time.perf_counter()
                    L.ctd_run_batches(ctx, c.cs, batch, count)
                    L.ctd_sync(ctx)
                    took.setdefault(name, []).append(time.perf_counter() - t0)
            # repeated runs of one configuration differ by 3 %
            assert min(took["kept"]) <= 1.10 * min(took["default"]), took
    finally:
        L.ctd_destroy(ctx)
