"""Dose, variance and sums as the readout kernels write them, against exact
integer arithmetic on the device tallies, from one voxel over the pieces that
the readout cuts a grid into."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from tests._helpers import random_phantom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _device_words(address, n):
    class A:
        __cuda_array_interface__ = dict(shape=(n,), typestr="<i8", data=(address, False),
                                        version=2)
    return torch.as_tensor(A(), device="cuda").cpu().numpy()


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 3, 5), (64, 32, 32), (41, 40, 40),
                                   (103, 97, 120)])
def test_readout_matches_exact_integers(ctx, shape):
    print(f"[gpu-test] readout {shape}", flush=True)
    wl = random_phantom(shape, 3, seed=5)
    wl.rho[0, 0, 0] = 0.0 if wl.rho.size > 1 else wl.rho[0, 0, 0]   # a voxel without mass
    with Case(ctx, wl) as c:
        L.ctd_run_batches(ctx, c.cs, 200_000, 5)
        L.ctd_sync(ctx)
        V = c.V
        s1, hi, lo, nb = c.tally()
        d1, d2 = L.ctd_tally_device(ctx, c.cs)
        assert nb == 5 and np.array_equal(s1, _device_words(d1, V))
        w = _device_words(d2, 2 * V).view(np.uint64)
        assert np.array_equal(lo, w[0::2]) and np.array_equal(hi, w[1::2])
        dose, var = c.dose()
        g = wl.grid
        mass = wl.rho.reshape(-1).astype(np.float64) * (g["dx"] * g["dy"] * g["dz"]) * 1e-3
        N = 1_000_000
        assert np.array_equal(dose == 0, (s1 == 0) | (mass == 0))
        rng = np.random.default_rng(1)
        for v in {0, V - 1, V // 2, int(np.argmax(s1)), *rng.integers(0, V, 300).tolist()}:
            if mass[v] == 0.0:
                assert dose[v] == 0.0 and var[v] == 0.0
                continue
            conv = 1.602176634e-16 / (16777216.0 * mass[v])
            num = nb * ((int(hi[v]) << 64) | int(lo[v])) - int(s1[v]) ** 2
            ref = num / (nb * nb * (nb - 1)) / (N / nb) ** 2 * conv * conv
            # a few roundings of 2^-53 each
            assert abs(dose[v] - int(s1[v]) / N * conv) <= 1e-15 * dose[v]
            assert abs(var[v] - ref) <= 4e-15 * abs(ref)
        # one plane alone
        only = np.full(V, np.nan)
        L.check(L.lib().ctd_read_dose(ctx, c.cs, None, L.ptr(only)), ctx)
        assert np.array_equal(only, var)
        n = C.c_uint32()
        L.check(L.lib().ctd_read_tally(ctx, c.cs, None, None, None, C.byref(n)), ctx)
        assert n.value == nb
