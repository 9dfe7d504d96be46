"""Coarse bound grid and parked photons of the deferred steps: the bytes reject
only fictitious collisions, and launches that use both leave the sums of
launches that read every collision's voxel, whatever the workgroup, the store's
size, the passes and the grid's cells."""
import os
import subprocess
import sys
from dataclasses import replace

import numpy as np
import pytest

from paper_1109_3266_amd import ctd as L
from paper_1109_3266_amd.session import Case
from synth import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1109_3266_amd", "csrc")


def test_coarse_bytes_bound_the_selection(tmp_path):
    """A word the byte rejects is fictitious in the float32 selection; a byte
    one lower (planted) is caught."""
    src = os.path.join(ROOT, "tests", "native", "share_check.cpp")

    def run(include, seed):
        exe = tmp_path / f"share_{seed}_{os.path.basename(include)}"
        subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", include, src,
                        "-o", str(exe)], check=True)
        return subprocess.run([str(exe), str(seed), "300"], check=True, capture_output=True,
                              text=True).stdout.split()

    for seed in (1, 7):
        out = run(CSRC, seed)
        assert out[0] == "ok" and int(out[1]) > 100_000, " ".join(out)
    header = open(os.path.join(CSRC, "ctd_bound.h")).read()
    old = "(unsigned char)x :"
    assert header.count(old) == 1
    d = tmp_path / "planted"
    d.mkdir()
    (d / "ctd_bound.h").write_text(header.replace(old, "(unsigned char)(x > 1 ? x - 1 : 0) :"))
    assert run(str(d), 1)[0] == "violation:"


@pytest.fixture(scope="module")
def ctx():
    h = L.ctd_create(0)
    yield h
    L.ctd_destroy(h)


def _noisy(nx, ny, nz, n_mat, seed):
    """A head-sized box of noisy ellipsoids in air (8-byte voxel records)."""
    base = W.head(scale=8)
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(*[np.linspace(-1, 1, n) if n > 1 else np.zeros(1)
                            for n in (nz, ny, nx)], indexing="ij")
    r = x * x + y * y + z * z
    mat = np.zeros((nz, ny, nx), np.uint8)
    for m in range(1, n_mat):
        mat[r < 0.8 * (n_mat - m) / n_mat] = m
    names = list(base.materials)[:n_mat]
    dens = np.array([W.ph.MATERIALS[m][0] for m in names])
    rho = dens[mat] * (1.0 + 0.02 * rng.standard_normal(mat.shape).clip(-3, 3))
    g = dict(nx=nx, ny=ny, nz=nz, dx=24.0 / nx, dy=24.0 / ny, dz=16.0 / nz, ox=-12.0, oy=-12.0,
             oz=-8.0)
    return replace(base, grid=g, materials=names, mat=mat, rho=rho.astype(np.float32))


def _sums(ctx, wl, n, tuning, log=False):
    with Case(ctx, wl) as c:
        L.ctd_set_tuning(ctx, c.cs, tuning)
        if log:
            L.ctd_debug_deposit_log(ctx, c.cs, 0, 1, 64)
        L.ctd_run_batches(ctx, c.cs, n, 2)
        s1, hi, lo, nb = c.tally()
        b, st = c.balance(), c.stats()
        assert b.q_incident == b.q_deposited + b.q_escaped
        return s1, hi, lo, nb, b.q_deposited, b.q_escaped, st.n_steps, st.n_real, st.n_deposits


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


# cells of one voxel (fewest, exactly 2560, one past it), ragged cells, thin
# grids; one history, part of a wave, several chunks; 1, 2 and 5 materials
@pytest.mark.gpu
@pytest.mark.parametrize("shape,n_mat,n", [
    ((8, 8, 8), 2, 1), ((16, 16, 10), 3, 63), ((17, 16, 10), 3, 20_000), ((20, 18, 1), 2, 5_000),
    ((37, 29, 41), 5, 60_000), ((65, 64, 33), 5, 200_000), ((300, 5, 7), 4, 30_000),
])
def test_parked_runs_match_plain_runs(ctx, shape, n_mat, n):
    print(f"[gpu-test] coarse grid {shape} {n_mat} materials {n}", flush=True)
    sys.stdout.flush()
    wl = _noisy(*shape, n_mat, seed=n)
    ref = _sums(ctx, wl, n, L.ctd_tuning(256, 5, 16, 1024, 0, 0, 16))
    # (block, waves per SIMD, refill, chunk, tally mode, bound block, defer_min)
    for t in [(256, 5, 16, 1024, 0, 2, 16), (256, 5, 64, 64, 0, 1, 64), (64, 5, 1, 64, 0, 2, 16),
              (512, 5, 24, 256, 0, 4, 1), (256, 8, 16, 1024, 0, 2, 32), (128, 2, 32, 128, 1, 2, 16),
              (256, 5, 16, 1024, 2, 2, 16), (256, 5, 16, 1024, 0, 2, 0)]:
        assert _same(_sums(ctx, wl, n, L.ctd_tuning(*t)), ref), t
    # with the event log nothing is parked and the coarse grid is not read
    assert _same(_sums(ctx, wl, n, L.ctd_tuning(256, 5, 16, 1024, 0, 2, 16), log=True), ref)
