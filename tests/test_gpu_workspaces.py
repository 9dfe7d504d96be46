"""The workspaces a context keeps between calls (deposit records, the tallies
and beamlets of shared launches, the gamma tool's block) are given back where
another allocation of the context finds no memory, and made anew afterwards."""
import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W
from tests._helpers import random_phantom

pytestmark = pytest.mark.gpu

ROOM = 40_000_000    # bytes; below what the runs here make the context keep


@pytest.fixture()
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _chains():
    wl = W.water_box_bowtie(scale=5)
    wl.geometry["fluence_chains"] = 100
    return wl


def _state(c):
    s1, hi, lo, nb = c.tally()
    b = c.balance()
    assert b.q_incident == b.q_deposited + b.q_escaped
    return s1, hi, lo, nb, b.q_deposited


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def _gamma(ctx):
    g = L.ctd_grid()
    g.nz, g.ny, g.nx = 20, 20, 20
    g.dx = g.dy = g.dz = 0.1
    ref = np.linspace(0.5, 1.0, 8000, dtype=np.float32)
    return L.ctd_gamma(ctx, g, ref, ref[::-1].copy(), 0.02, 0.2, 0.3)[0]


@pytest.mark.parametrize("kind", ["load", "macro", "tuning", "beamlets", "log", "autotune"])
def test_workspaces_give_way(ctx, kind):
    print(f"[gpu-test] workspaces give way to {kind}", flush=True)
    wl = W.tiny()
    with Case(ctx, wl) as a, Case(ctx, wl) as b, Case(ctx, _chains()) as m:
        before = _gamma(ctx)
        L.ctd_run_batches(ctx, a.cs, 400_000, 3)
        assert L.ctd_debug_launches(ctx) == (1, 1)          # shared, with records
        L.ctd_debug_limits(ctx, memory_bytes=ROOM)
        if kind in ("load", "macro"):
            other = random_phantom((6, 7, 8), 4, seed=2)
            Case(ctx, other, tracking=L.CTD_TRACK_MACRO if kind == "macro" else None).close()
        elif kind == "tuning":
            L.ctd_set_tuning(ctx, b.cs, L.ctd_tuning(256, 5, 16, 1024, 1, 2, 16))
        elif kind == "beamlets":
            L.ctd_run_batches(ctx, m.cs, 1000, 1)
        elif kind == "log":
            L.ctd_debug_deposit_log(ctx, b.cs, 0, 10, 1000)
        else:
            L.ctd_autotune(ctx, b.cs, 1000)
        L.ctd_debug_limits(ctx)
        # the workspaces come back where launches want them
        n0, r0 = L.ctd_debug_launches(ctx)
        L.ctd_run_batches(ctx, a.cs, 400_000, 3)
        n1, r1 = L.ctd_debug_launches(ctx)
        assert (n1 - n0, r1 - r0) == (1, 1)
        for _ in range(6):
            L.ctd_run_batches(ctx, b.cs, 400_000, 1)
        _same(_state(a), _state(b))
        assert np.array_equal(_gamma(ctx), before)
