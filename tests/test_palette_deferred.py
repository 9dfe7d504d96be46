"""Piecewise-constant phantoms of which few collisions deposit run with the
deferred steps, their voxel indices as the bound grid: the same sums as the
plain steps (bound_block = 0) leave, solo and in a batched round with plain
and record phantoms."""
import sys
from dataclasses import replace

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


def _body(nx, ny, nz, levels, bone, seed):
    """Ellipsoids in air, one density per material and level; bone makes most
    collisions fictitious."""
    base = W.head(scale=8)
    names = ["air", "soft_tissue"] + (["cortical_bone"] if bone else [])
    z, y, x = np.meshgrid(*[np.linspace(-1, 1, n) if n > 1 else np.zeros(1)
                            for n in (nz, ny, nx)], indexing="ij")
    r = x * x + y * y + z * z
    mat = (r < 0.7).astype(np.uint8)
    if bone:
        mat[r < 0.02] = 2
    dens = np.array([W.ph.MATERIALS[m][0] for m in names])
    step = np.random.default_rng(seed).integers(0, levels, mat.shape)
    rho = dens[mat] * (1.0 - 0.3 * step / max(levels, 1))
    if levels == 85:   # 3 x 85 entries, and the 256th
        rho.flat[0] *= 1.1
    g = dict(nx=nx, ny=ny, nz=nz, dx=24.0 / nx, dy=24.0 / ny, dz=16.0 / nz, ox=-12.0, oy=-12.0,
             oz=-8.0)
    return replace(base, grid=g, materials=names, mat=mat, rho=rho.astype(np.float32))


def _read(c):
    s1, hi, lo, nb = c.tally()
    b, st = c.balance(), c.stats()
    assert b.q_incident == b.q_deposited + b.q_escaped
    return s1, hi, lo, nb, b.q_escaped, st.n_steps, st.n_real, st.n_deposits


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def _solo(ctx, wl, n, bound, log=False):
    with Case(ctx, wl) as c:
        L.ctd_set_tuning(ctx, c.cs, L.ctd_tuning(256, 5, 16, 1024, 0, bound, 16))
        if log:
            L.ctd_debug_deposit_log(ctx, c.cs, 0, 1, 64)
        L.ctd_run_batches(ctx, c.cs, n, 2)
        return _read(c)


# few and all 256 palette entries (the last index is also the mixed class's),
# ragged grids, without bone (plain steps either way), one history and many
@pytest.mark.parametrize("shape,levels,bone,n", [
    ((16, 16, 10), 1, True, 1), ((33, 29, 17), 1, True, 50_000), ((40, 40, 24), 85, True, 50_000),
    ((48, 40, 33), 3, True, 400_000), ((33, 29, 17), 2, False, 50_000),
])
def test_palette_runs_match_plain_runs(ctx, shape, levels, bone, n):
    print(f"[gpu-test] palette deferred {shape} {levels} {bone} {n}", flush=True)
    sys.stdout.flush()
    wl = _body(*shape, levels, bone, seed=n)
    ref = _solo(ctx, wl, n, 0)
    for bound in (1, 2, 4):
        assert _same(_solo(ctx, wl, n, bound), ref), bound
    assert _same(_solo(ctx, wl, n, 2, log=True), ref)


# one case after another (mode 0) and rounds over all cases (mode 1), in which
# the two deferred cases share launches and workgroups change between them
@pytest.mark.parametrize("mode", [0, 1])
def test_run_of_all_three_phantom_kinds(ctx, mode):
    print(f"[gpu-test] deferred palette, plain palette and records, mode {mode}", flush=True)
    sys.stdout.flush()
    wls = [_body(33, 29, 17, 2, True, 1), _body(24, 24, 20, 2, False, 2), W.head(scale=8)]
    n = [30_000, 40_001, 20_000]

    def run(members, bound, mode):
        cases = [Case(ctx, wls[i]) for i in members]
        try:
            for c in cases:
                L.ctd_set_tuning(ctx, c.cs, L.ctd_tuning(256, 5, 16, 1024, mode, bound, 16))
            for _ in range(2):
                L.ctd_run_many(ctx, [c.cs for c in cases], [n[i] for i in members])
            return [_read(c) for c in cases]
        finally:
            for c in cases:
                c.close()

    for i, got in enumerate(run([0, 1, 2], 2, mode)):
        assert _same(run([i], 0, 0)[0], got), i
