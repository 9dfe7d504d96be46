"""Gamma index on a grid whose voxels are far smaller than a lattice step: the
step's cell lies past the end of the int range, and the interpolation takes the
grid's outermost dose on the side the step goes to."""
import numpy as np
import pytest

from oracle import gamma as OG
from paper_1109_3266_amd import ctd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_lattice_steps_beyond_every_cell(axis):
    print(f"[gpu-test] gamma lattice beyond the cells, axis {axis}", flush=True)
    shape = [2, 3, 4]
    shape[axis] = 1500
    d = [0.3, 0.3, 0.3]                    # z, y, x
    d[axis] = 1e-11
    rng = np.random.default_rng(9)
    ref = np.ones(shape, np.float32)
    ev = (1.5 + 0.1 * rng.standard_normal(shape)).astype(np.float32)
    edge = [slice(None)] * 3
    edge[axis] = slice(-1, None)
    ev[tuple(edge)] = 1.0                  # the far end matches, the near one does not
    g = L.ctd_grid()
    g.nz, g.ny, g.nx = shape
    g.dz, g.dy, g.dx = d
    kw = dict(dose_tol=0.02, dta_cm=0.1, region_min=0.3, gamma_cap=2.0, substeps=3)
    want, n_region, _ = OG.gamma_index(ref, ev, (d[2], d[1], d[0]), **kw)
    ctx = L.ctd_create(0)
    try:
        got, n, _ = L.ctd_gamma(ctx, g, ref, ev, **kw)
    finally:
        L.ctd_destroy(ctx)
    assert n == n_region
    assert np.allclose(got.reshape(shape), want, rtol=1e-6, atol=1e-6)
