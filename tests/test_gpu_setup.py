"""Set-up kernels: the palette found on the device at the edges of its 256
records, through the sums that follow from it, and the macro cells' maxima at
edges of cells."""
import math

import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from tests._helpers import random_phantom, slab_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _sums(ctx, wl, **kw):
    tuning = kw.pop("tuning", None)
    with Case(ctx, wl, **kw) as c:
        if tuning is not None:
            L.ctd_set_tuning(ctx, c.cs, tuning)
        L.ctd_run_batches(ctx, c.cs, 50_000, 2)
        s1, hi, lo, nb = c.tally()
        b = c.balance()
        assert b.q_incident == b.q_deposited + b.q_escaped and int(s1.sum()) == b.q_deposited
        return s1, hi, lo


# distinct records: one, a few, the most a palette holds, one more (8-byte
# layout), and a constant phantom with noise in one corner only, which the
# sampled look does not see
@pytest.mark.parametrize("levels,corner", [(1, False), (3, False), (255, False), (256, False),
                                           (257, False), (300, True), (20_000, True)])
def test_palette_edges(ctx, levels, corner):
    print(f"[gpu-test] palette of {levels} records, corner={corner}", flush=True)
    wl = random_phantom((24, 33, 41), 2, seed=9)
    n = wl.rho.size
    rng = np.random.default_rng(levels)
    mat = np.zeros(n, np.uint8)
    rho = np.ones(n, np.float32)
    value = (0.9 + 0.2 * np.arange(levels) / max(1, levels)).astype(np.float32)
    if corner:
        rho[-levels:] = value
    else:
        rho[rng.permutation(n)[:levels]] = value
        rho[rho == 1.0] = value[0]
    rho[7] = -0.0 if not corner and levels == 3 else rho[7]   # packed as +0
    wl.mat, wl.rho = mat.reshape(wl.mat.shape), rho.reshape(wl.rho.shape)
    a = _sums(ctx, wl)
    # the same densities with half of the voxels in a second material of the
    # same cross sections: other records and another layout, the same dose
    two = wl.mu_rho().copy()
    two[1] = two[0]
    b_mat = mat.copy()
    b_mat[rng.permutation(n)[: n // 2]] = 1
    wl.mat = b_mat.reshape(wl.mat.shape)
    wl.materials = [wl.materials[0]] * 2
    b = _sums(ctx, wl, mu_rho=two)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    # with the bound grid off the 8-byte layout takes the plain step
    c = _sums(ctx, wl, mu_rho=two, tuning=L.ctd_tuning(256, 5, 16, 1024, 0, 0, 16))
    for x, y in zip(a, c):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("cell,plane", [(7, 6), (8, 7), (8, 8), (9, 16), (16, 15), (64, 16)])
def test_macro_cells_hold_their_edge_voxels(ctx, cell, plane):
    """One plane of bone in water at the last or first plane of a cell, cells
    that end past the grid: a cell majorant without it would let collisions
    there go missing.  Unscattered transmission of a 60 keV pencil, exp(-sum
    mu_i L_i), within 4.5 standard deviations of 1e7 histories."""
    print(f"[gpu-test] macro cell {cell}, bone at plane {plane}", flush=True)
    layers = [("water", 1.0, plane), ("cortical_bone", 1.85, 1), ("water", 1.0, 17 - plane)]
    wl = slab_workload([x for x in layers if x[2]], e_kev=60.0, n_hist=10_000_000, seed=17,
                       nxy=5, dz=0.5)
    tab = wl.mu_rho().astype(np.float64)
    j = int(round(60.0 - wl.e0))
    mu_l = sum(r * tab[wl.materials.index(m), j, :].sum() * n * 0.5 for m, r, n in layers)
    p = math.exp(-mu_l)
    with Case(ctx, wl, tracking=L.CTD_TRACK_MACRO, macro_cell=cell) as c:
        c.run(wl.n_histories)
        frac = c.balance().n_unscattered / wl.n_histories
    assert abs(frac - p) < 4.5 * math.sqrt(p * (1 - p) / wl.n_histories)
