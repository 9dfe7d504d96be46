"""A context on the per-thread default stream: the readouts' helper threads,
whose per-thread stream is another one, copy what the caller's stream has
computed."""
import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W

pytestmark = pytest.mark.gpu

PER_THREAD = 2      # hipStreamPerThread


@pytest.fixture()
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


@pytest.mark.parametrize("shape", [(3, 4, 5), (96, 100, 104)])
def test_gamma_on_the_per_thread_stream(ctx, shape):
    print(f"[gpu-test] per-thread stream, gamma {shape}", flush=True)
    rng = np.random.default_rng(3)
    g = L.ctd_grid()
    g.nz, g.ny, g.nx = shape
    g.dx = g.dy = g.dz = 0.1
    want, got = [], []
    for out, stream in ((want, None), (got, PER_THREAD)):
        L.ctd_set_stream(ctx, stream)
        rng = np.random.default_rng(3)
        for _ in range(3):       # other doses each time: no earlier result fits
            ref = (1.0 + 0.05 * rng.standard_normal(shape)).astype(np.float32)
            ev = (ref * (1.0 + 0.03 * rng.standard_normal(shape))).astype(np.float32)
            out.append(L.ctd_gamma(ctx, g, ref, ev, 0.02, 0.2, 0.3))
    L.ctd_set_stream(ctx, None)
    for a, b in zip(want, got):
        assert np.array_equal(a[0], b[0]) and a[1:] == b[1:]


def test_run_and_readout_on_the_per_thread_stream(ctx):
    print("[gpu-test] per-thread stream, run and readout", flush=True)
    wl = W.water_cbct(scale=2)
    with Case(ctx, wl) as a, Case(ctx, wl) as b:
        a.run(200_000)
        want = a.dose() + a.tally()
        L.ctd_set_stream(ctx, PER_THREAD)
        b.run(200_000)
        got = b.dose() + b.tally()
        L.ctd_set_stream(ctx, None)
        for x, y in zip(want, got):
            assert np.array_equal(x, y)
