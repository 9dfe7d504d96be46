"""Gamma index next to doses that are not finite: a lattice point whose
interpolant is formed with such a dose (weight 0 included) is left out, the
voxel's own centre like any other, at every voxel of the grid."""
import numpy as np
import pytest

from oracle import gamma as OG
from paper_1109_3266_amd import ctd as L

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _expected(ref, ev, d, dose_tol, dta, region, cap, sub):
    """The oracle's points, each left out where its interpolant is not a
    number."""
    R, E = ref.astype(np.float64), ev.astype(np.float64)
    iz, iy, ix = np.nonzero(R > region)
    best = np.full(iz.shape, cap * cap)
    h = dta / sub
    with np.errstate(invalid="ignore"):
        for i, j, k in OG.lattice(dta, cap, sub):
            de = OG.trilinear(E, ix + i * h / d, iy + j * h / d, iz + k * h / d)
            far = (i * i + j * j + k * k) / (sub * sub)
            best = np.fmin(best, far + (R[iz, iy, ix] - de) ** 2 / dose_tol ** 2)
    out = np.full(R.shape, -1.0)
    out[iz, iy, ix] = np.sqrt(best)
    return out


# lattice steps of 0.5 and 0.75 voxels (exact in binary, so every point's cell
# is certain); the bad dose inside, on a face and in each kind of corner
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("dta,shape,at", [
    (0.5, (7, 6, 9), (3, 3, 4)), (0.75, (7, 6, 9), (0, 0, 0)), (0.5, (5, 6, 70), (4, 5, 69)),
    (0.75, (5, 6, 70), (2, 0, 69)), (0.5, (1, 6, 70), (0, 3, 40)),
])
def test_gamma_beside_non_finite_doses(ctx, dta, shape, at, bad):
    print(f"[gpu-test] gamma beside {bad} at {at} of {shape}", flush=True)
    rng = np.random.default_rng(6)
    ref = (1.0 + 0.05 * rng.standard_normal(shape)).astype(np.float32)
    ev = ref.copy()                      # every voxel's own centre matches best
    ev[at] = bad
    d = 0.25
    g = L.ctd_grid()
    g.nz, g.ny, g.nx = shape
    g.dx = g.dy = g.dz = d
    got, n_region, _ = L.ctd_gamma(ctx, g, ref, ev, 0.02, dta, 0.3, gamma_cap=2.0, substeps=4)
    want = _expected(ref, ev, d, 0.02, dta, 0.3, 2.0, 4)
    assert n_region == ref.size
    assert np.allclose(got.reshape(shape), want, rtol=1e-6, atol=1e-6)
    assert (want > 1e-3).sum() >= 1      # some centre does not count
