"""The gamma kernel's cells against the brute-force oracle where they can go
wrong: grids of one and two voxels per axis (every cell at a border), lattice
steps that hit voxel centres, voxels far smaller and far larger than the search
radius, and device arrays; non-finite doses leave the finite voxels' search
as the oracle's."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import gamma as OG
from paper_1109_3266_amd import ctd as L

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _g(shape, d):
    g = L.ctd_grid()
    g.nz, g.ny, g.nx = shape
    g.dx, g.dy, g.dz = d
    return g


def _check(ctx, shape, d, ref, ev, **kw):
    with np.errstate(invalid="ignore"):
        go, nr, npass = OG.gamma_index(ref, ev, d, **kw)
    gg, nr_g, np_g = L.ctd_gamma(ctx, _g(shape, d), ref, ev, **kw)
    assert nr_g == nr
    # the last rounding to float32, and FP64 sums in another order
    assert np.allclose(gg.reshape(shape), go, rtol=1e-6, atol=1e-6)
    assert abs(np_g - npass) <= int(np.count_nonzero(np.abs(go ** 2 - 1.0) < 1e-9))
    return gg, nr, npass


@pytest.mark.parametrize("shape,d,dta,cap,sub", [
    ((1, 1, 1), (0.1, 0.1, 0.1), 0.2, 2.0, 5), ((2, 1, 3), (0.1, 0.3, 0.1), 0.3, 2.0, 3),
    ((2, 2, 2), (0.02, 0.02, 0.02), 0.1, 1.5, 4),          # cells of at most one point
    ((9, 8, 70), (0.1, 0.1, 0.1), 0.2, 2.0, 4),            # steps on voxel centres
    ((5, 6, 7), (3.0, 2.0, 1.0), 0.2, 4.0, 7),             # one cell per octant
])
def test_cells_match_oracle(ctx, shape, d, dta, cap, sub):
    print(f"[gpu-test] gamma cells {shape} {d}", flush=True)
    rng = np.random.default_rng(4)
    ref = (1.0 + 0.05 * rng.standard_normal(shape)).astype(np.float32)
    ev = (ref * (1.0 + 0.03 * rng.standard_normal(shape))).astype(np.float32)
    kw = dict(dose_tol=0.02, dta_cm=dta, region_min=0.3, gamma_cap=cap, substeps=sub)
    g, nr, npass = _check(ctx, shape, d, ref, ev, **kw)
    # the same from device arrays
    r, e = torch.from_numpy(ref).cuda(), torch.from_numpy(ev).cuda()
    out = torch.empty(ref.size, device="cuda")
    torch.cuda.synchronize()
    p = L.ctd_gamma_params(0.02, dta, 0.3, cap, sub, 0)
    a, b = C.c_uint64(), C.c_uint64()
    L.check(L.lib().ctd_gamma(ctx, C.byref(_g(shape, d)), L.ptr(r), L.ptr(e), L.CTD_MEM_DEVICE,
                              C.byref(p), L.ptr(out), C.byref(a), C.byref(b)), ctx)
    assert (a.value, b.value) == (nr, npass)
    assert np.array_equal(out.cpu().numpy(), g)


def test_plateaus_and_non_finite_doses(ctx):
    print("[gpu-test] gamma plateaus and non-finite doses", flush=True)
    shape, d = (6, 7, 66), (0.1, 0.1, 0.1)
    ref, ev = np.ones(shape, np.float32), np.ones(shape, np.float32)
    ev[:, :, 30:] = 1.5
    kw = dict(dose_tol=0.02, dta_cm=0.2, region_min=0.3, gamma_cap=2.0, substeps=5)
    _check(ctx, shape, d, ref, ev, **kw)
    for bad in (np.nan, np.inf, -np.inf):
        for at in ((0, 0, 0), (3, 3, 33), (5, 6, 65)):
            e2 = ev.copy()
            e2[at] = bad
            r2 = ref.copy()
            r2[2, 2, 2] = bad
            with np.errstate(invalid="ignore"):
                go, nr, _ = OG.gamma_index(r2, e2, d, **kw)
            gg, nr_g, _ = L.ctd_gamma(ctx, _g(shape, d), r2, e2, **kw)
            assert nr_g == nr
            far = np.ones(shape, bool)      # beyond the search radius of the bad dose
            z, y, x = np.indices(shape)
            far &= (z - at[0]) ** 2 + (y - at[1]) ** 2 + (x - at[2]) ** 2 > 6 ** 2
            far[2, 2, 2] = False
            assert np.allclose(gg.reshape(shape)[far], go[far], rtol=1e-6, atol=1e-6)
            g = gg.reshape(shape)[~far]
            assert np.all((g == -1.0) | ((g >= 0.0) & (g <= 2.0)))
