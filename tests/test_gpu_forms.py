"""Forms of the kernels that a launch chooses by the size of its work, at the
sizes where one form ends and the next begins.  The particles' streams fix every
history, so the physics events must be the same whole numbers and the doses the
same up to the order of the FP64 tally additions (a sum of n terms reorders to
within n ulps; voxel sums here have below 1e4 terms: 1e-12)."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1107_3355_amd import gdpm as G
from paper_1107_3355_amd import inputs as I
from tests.gpu_common import balance, gpu_run, physics_events
from tests.test_gpu_parity import check_statistics

pytestmark = pytest.mark.gpu
MATS = I.MATERIALS


def _same(a, b):
    assert physics_events(a) == physics_events(b)
    assert a["interactions"] == b["interactions"]
    np.testing.assert_allclose(a["dose"], b["dose"], rtol=1e-12, atol=1e-12 * b["dose"].max())


# a chain of Metropolis beamlets gets as many lanes of the source pass as it has
# steps in a segment (16,384 chains): 1, 2, 4, 16 and 64 lanes, with steps left over
@pytest.mark.parametrize("per_pass", [1_000, 16_384 * 2 + 1, 16_384 * 5 + 77, 16_384 * 17, 16_384 * 70 + 3])
def test_metropolis_lanes(gctx, per_pass):
    ph = I.ct_phantom((32, 32, 16), (1.5, 1.5, 2.0))
    src = I.Source(I.PHOTON, I.triangular_spectrum(), I.imrt_plan(ph, nb=6), beamlet_sampler=1, spectrum_strata=5)
    n = min(1_300_007, 12 * per_pass)
    kw = dict(n_hist=n, seed=5, n_batches=2, hist0=123)
    c = G.Context(0, opts=f'{{"pass_histories": {per_pass}}}', materials=MATS)
    try:
        a = gpu_run(c, ph, src, **kw)
    finally:
        c.close()
    # the reference walks the chains one step at a time: 8 histories per chain and pass at most
    c = G.Context(0, opts='{"pass_histories": 16383}', materials=MATS)
    try:
        b = gpu_run(c, ph, src, **kw)
    finally:
        c.close()
    _same(a, b)
    assert balance(a) < 1e-12


# units of 64 histories of the source pass: a full one, one short, one over, and
# the copies of a split history (written one by one)
@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("n", [63, 64, 65, 129, 4097])
def test_source_units(gctx, n, split):
    w = I.water_cube_2mev(n)
    a = gpu_run(gctx, w.phantom, w.source, n_hist=n, seed=3, n_batches=2, want_hist=True, split_log2=split)
    b = gpu_run(gctx, w.phantom, w.source, n_hist=n, seed=3, n_batches=3, want_hist=True, split_log2=split)
    # every history is there once: its energy is the source's, whichever segment it came in
    np.testing.assert_allclose(a["hist"].sum(axis=1), 2.0, rtol=1e-12)
    np.testing.assert_allclose(a["hist"], b["hist"], rtol=0, atol=1e-12)
    assert a["histories"] == n and balance(a) < 1e-12


# the statistics hold ten batches in registers, read up to 32 normalisations from
# the kernel's arguments and more from memory
@pytest.mark.parametrize("nb", [2, 9, 10, 11, 32, 33, 70])
def test_statistics_batches(gctx, nb):
    w = I.water_cube_2mev(20_000)
    g = gpu_run(gctx, w.phantom, w.source, n_hist=20_000, seed=8, n_batches=nb, want_batches=True)
    check_statistics(g, w.phantom, 20_000, nb=nb)


# host outputs travel in 1 MiB chunks, at most 32 at a time: less than one, a few, more than 32
@pytest.mark.parametrize("side", [20, 64, 140])
def test_host_outputs(gctx, side):
    ph = I.homogeneous((side, side, side), (16.0 / side,) * 3, I.ID_WATER, 1.0)
    src = I.Source(I.PHOTON, I.mono(2.0), [I.parallel_beam_z(ph, 5.0)])
    g = gpu_run(gctx, ph, src, n_hist=3_000, seed=2, n_batches=2, want_batches=True)
    check_statistics(g, ph, 3_000, nb=2)


# the electron pass sums a particle's deposits per brick of the tally, two voxels wide
# along up to two axes with an even number of voxels; with the batches as an output the
# tally stays in plain order and every deposit is added by itself
@pytest.mark.parametrize("opts", ['{}', '{"lds_tables": 0}', '{"fused_passes": 1}',
                                  '{"rebin_photons": 1, "rebin_electrons": 1}'])
@pytest.mark.parametrize("n", [(8, 10, 12), (9, 10, 12), (8, 11, 12), (8, 10, 13), (9, 11, 12), (8, 11, 13),
                               (9, 11, 13), (1, 1, 2), (2, 1, 1), (1, 30, 1)])
def test_tally_bricks(n, opts):
    rng = np.random.default_rng(sum(n))
    d = (0.3, 0.2, 0.25) if n[0] % 2 else (0.2, 0.3, 0.25)
    ph = I.Phantom(*n, *d, rng.integers(1, 4, n[::-1]).astype(np.uint8), rng.uniform(0.3, 1.6, n[::-1]).astype(np.float32))
    src = I.Source(I.ELECTRON, I.mono(6.0), [I.parallel_beam_z(ph, min(n[0] * d[0], n[1] * d[1]))])
    kw = dict(n_hist=20_000, seed=11, n_batches=3)
    c = G.Context(0, opts=opts, materials=MATS)
    try:
        a = gpu_run(c, ph, src, **kw)
        b = gpu_run(c, ph, src, want_batches=True, **kw)
    finally:
        c.close()
    _same(a, b)
    np.testing.assert_allclose(a["sigma"], b["sigma"], rtol=1e-9, atol=1e-12 * b["dose"].max())
    assert balance(a) < 1e-12
    check_statistics(b, ph, 20_000, nb=3)


# tables that leave no room for the brick sums beside them (6 materials), or that
# are not staged (8)
@pytest.mark.parametrize("n_mat", [5, 6, 7, 8])
def test_more_materials(n_mat):
    mats = (list(MATS) + list(MATS))[:n_mat]
    n, d = (16, 16, 20), (0.5, 0.5, 0.5)
    mat = (np.arange(16 * 16 * 20).reshape(n[::-1]) % n_mat).astype(np.uint8)
    ph = I.Phantom(*n, *d, mat, np.ones(n[::-1], np.float32))
    src = I.Source(I.PHOTON, I.mono(6.0), [I.parallel_beam_z(ph, 4.0)])
    res = []
    for opts in ('{}', '{"lds_tables": 0, "waves_per_cu": 4}'):
        c = G.Context(0, opts=opts, materials=mats)
        try:
            res.append(gpu_run(c, ph, src, n_hist=20_000, seed=4, n_batches=2))
        finally:
            c.close()
    _same(*res)


# a pass with 16 records or more per lane of its 16 wavefronts per CU runs them all,
# one with fewer runs 12 (3 and 4 here): below, at and above the line in one run
def test_wide_passes():
    w = I.water_cube_2mev(2_600_000)
    res = []
    for opts in ('{"waves_per_cu": 3}', '{"waves_per_cu": 12, "pass_histories": 100000}'):
        c = G.Context(0, opts=opts, materials=MATS)
        try:
            res.append(gpu_run(c, w.phantom, w.source, n_hist=2_600_000, seed=4, n_batches=2))
        finally:
            c.close()
    a, b = res
    assert physics_events(a) == physics_events(b)
    rtol = 2 * max(sum(r["deposits"]) for r in res) * np.finfo(float).eps   # any order of all deposits
    np.testing.assert_allclose(a["dose"], b["dose"], rtol=rtol, atol=rtol * b["dose"].max())


# several jobs: 8 records per lane in each of them on average
@pytest.mark.parametrize("n", [400_000, 1_500_000])
def test_wide_passes_of_jobs(n):
    w = I.water_cube_2mev(n)
    kw = dict(n_hist=n, seed=4, n_batches=2)
    c = G.Context(0, opts='{"waves_per_cu": 3}', materials=MATS)
    try:
        ph, src = c.phantom(w.phantom), c.source(w.source)
        a = c.run_batch([(ph, src, dict(kw, job_id=k)) for k in range(2)])
        b = [c.run(ph, src, **dict(kw, job_id=k)) for k in range(2)]
    finally:
        c.close()
    for x, y in zip(a, b):
        rtol = 2 * max(sum(r["deposits"]) for r in b) * np.finfo(float).eps   # any order of all deposits
        np.testing.assert_allclose(x["dose"], y["dose"], rtol=rtol, atol=rtol * y["dose"].max())


# photon passes with 4 records or more per lane park the photons that interact (here
# with one wavefront per CU: from 65,536), shorter ones let them wait in their lanes:
# absorption alone, scattering, pairs; one particle per wavefront; several jobs
@pytest.mark.parametrize("opts", ['{"waves_per_cu": 1}', '{"waves_per_cu": 1, "lds_tables": 0}',
                                  '{"waves_per_cu": 1, "fused_passes": 1}', '{"waves_per_cu": 2, "solo_lanes": 1}',
                                  '{"waves_per_cu": 1, "rebin_photons": 1}'])
@pytest.mark.parametrize("e", [0.06, 1.0, 15.0])
def test_photon_pool(e, opts):
    ph = I.homogeneous((20, 20, 20), (1.0,) * 3, I.ID_BONE, 1.85)
    src = I.Source(I.PHOTON, I.mono(e), [I.parallel_beam_z(ph, 10.0)])
    n = 20_000 if "solo" in opts else 150_000
    res = []
    for o in (opts, '{"pass_histories": 3000}'):
        c = G.Context(0, opts=o, materials=MATS)
        try:
            res.append(gpu_run(c, ph, src, n_hist=n, seed=6, n_batches=2))
        finally:
            c.close()
    a, b = res
    assert physics_events(a) == physics_events(b) and a["interactions"] == b["interactions"]
    rtol = 2 * max(sum(r["deposits"]) for r in res) * np.finfo(float).eps   # any order of all deposits
    np.testing.assert_allclose(a["dose"], b["dose"], rtol=rtol, atol=rtol * b["dose"].max())
    assert balance(a) < 1e-12


def test_photon_pool_jobs():
    ph = I.homogeneous((20, 20, 20), (1.0,) * 3, I.ID_WATER, 1.0)
    src = I.Source(I.PHOTON, I.mono(6.0), [I.parallel_beam_z(ph, 10.0)])
    kws = [dict(n_hist=n, seed=6, n_batches=2, job_id=k) for k, n in enumerate((90_000, 3_000, 120_000, 64, 70_001))]
    c = G.Context(0, opts='{"waves_per_cu": 1}', materials=MATS)
    try:
        p, s = c.phantom(ph), c.source(src)
        many = c.run_batch([(p, s, kw) for kw in kws])
        one = [c.run(p, s, **kw) for kw in kws]
    finally:
        c.close()
    for a, b in zip(many, one):
        rtol = 2 * sum(b["deposits"]) * np.finfo(float).eps
        np.testing.assert_allclose(a["dose"], b["dose"], rtol=rtol, atol=rtol * b["dose"].max())


# both passes in one launch, with the wavefronts it has by default: few and many records
# per lane (the hand-off at the tail of a long pass), queues read as they are and
# through the permutation, all kinds of shares, and tables with less room beside them
@pytest.mark.parametrize("n_mat,opts", [(4, ''), (4, ', "photon_waves": 0'), (4, ', "photon_waves": 12'), (5, ''), (6, ''),
                                        (4, ', "rebin_photons": 1, "rebin_electrons": 1'),
                                        (4, ', "rebin_photons": 1'), (4, ', "waves_per_cu": 5')])
@pytest.mark.parametrize("n", [3_000, 1_000_000])
def test_fused_passes(n, n_mat, opts):
    mats = (list(MATS) + list(MATS))[:n_mat]
    rng = np.random.default_rng(n_mat)
    shape = (20, 18, 15)
    ph = I.Phantom(*shape, 0.6, 0.5, 0.8, rng.integers(0, n_mat, shape[::-1]).astype(np.uint8),
                   rng.uniform(0.3, 1.6, shape[::-1]).astype(np.float32))
    src = I.Source(I.PHOTON, I.mono(6.0), [I.parallel_beam_z(ph, 6.0)])
    res = []
    for o in ('{"fused_passes": 1' + opts + '}', '{}'):
        c = G.Context(0, opts=o, materials=mats)
        try:
            res.append(gpu_run(c, ph, src, n_hist=n, seed=4, n_batches=2))
        finally:
            c.close()
    a, b = res
    assert a["t_photon_s"] == 0 and a["t_electron_s"] == 0 and a["t_kernel_s"] > 0   # one launch for both
    assert b["t_photon_s"] > 0 and b["t_electron_s"] > 0
    assert physics_events(a) == physics_events(b) and a["interactions"] == b["interactions"]
    rtol = 2 * max(sum(r["deposits"]) for r in res) * np.finfo(float).eps   # any order of all deposits
    np.testing.assert_allclose(a["dose"], b["dose"], rtol=rtol, atol=rtol * b["dose"].max())
    assert balance(a) < 1e-12


# the forms without staged tables take more than 64 KB of LDS too: in a process of their
# own, where no other context has asked for it
def test_unstaged_tables_alone(gctx):
    code = ("from paper_1107_3355_amd import gdpm as G, inputs as I\n"
            "from tests.gpu_common import gpu_run, physics_events\n"
            "w = I.water_cube_2mev(40_000)\n"
            "c = G.Context(0, opts='{\"lds_tables\": 0}', materials=I.MATERIALS)\n"
            "r = gpu_run(c, w.phantom, w.source, n_hist=40_000, seed=9)\n"
            "print(physics_events(r))\n")
    out = subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                         capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr
    w = I.water_cube_2mev(40_000)
    assert out.stdout.strip() == str(physics_events(gpu_run(gctx, w.phantom, w.source, n_hist=40_000, seed=9)))


# electron passes of many records with tables that leave room for 16, 13 (5 materials)
# and no wavefronts with brick sums
@pytest.mark.parametrize("n_mat", [4, 5, 6])
def test_wide_passes_with_more_materials(n_mat):
    mats = (list(MATS) + list(MATS))[:n_mat]
    shape, n = (20, 20, 20), 4_500_000
    ph = I.Phantom(*shape, 0.1, 0.1, 0.1, (np.arange(8000).reshape(shape) % n_mat).astype(np.uint8),
                   np.ones(shape, np.float32))
    src = I.Source(I.ELECTRON, I.mono(0.9), [I.parallel_beam_z(ph, 2.0)])
    res = []
    for opts in ('{}', '{"lds_tables": 0, "waves_per_cu": 12, "pass_histories": 500000}'):
        c = G.Context(0, opts=opts, materials=mats)
        try:
            res.append(gpu_run(c, ph, src, n_hist=n, seed=4, n_batches=2))
        finally:
            c.close()
    a, b = res
    assert physics_events(a) == physics_events(b) and a["interactions"] == b["interactions"]
    rtol = 2 * max(sum(r["deposits"]) for r in res) * np.finfo(float).eps   # any order of all deposits
    np.testing.assert_allclose(a["dose"], b["dose"], rtol=rtol, atol=rtol * b["dose"].max())
    assert balance(a) < 1e-9


# the slots that wavefronts reserve and leave unused, 128 each on average with 12 per CU: a
# queue of 2^23 records has room for them beside one electron of each of 7.93e6 photons
# (0.39e6 slots), with 16 wavefronts as well
def test_reserved_slots_of_wide_passes():
    n = 7_930_000
    ph = I.homogeneous((16, 16, 16), (1.0,) * 3, I.ID_BONE, 2.0e4)
    src = I.Source(I.PHOTON, I.mono(0.3), [I.parallel_beam_z(ph, 8.0)])
    c = G.Context(0, opts=f'{{"ring_capacity_log2": 23, "pass_histories": {n}}}', materials=MATS)
    try:
        r = gpu_run(c, ph, src, n_hist=n, seed=2, n_batches=2,
                    flags=G.NO_COMPTON | G.NO_PAIR | G.NO_MOLLER | G.NO_BREMS, want_dose=False)
    finally:
        c.close()
    assert r["events"]["pushes"] == r["interactions"]["photo"] > 0.99 * n
    assert balance(r) < 1e-9


# 64 lanes for a chain: a segment of 70 steps of every chain and a few histories more, and
# the next one, whose chains start at other steps
def test_metropolis_64_lanes(gctx):
    n, chains = 2_300_007, 16_384
    segment = -(-n // 2)                  # two batches
    lanes = 1
    while lanes < 64 and 2 * lanes <= segment // chains:
        lanes *= 2
    assert lanes == 64
    ph = I.ct_phantom((32, 32, 16), (1.5, 1.5, 2.0))
    src = I.Source(I.PHOTON, I.triangular_spectrum(), I.imrt_plan(ph, nb=6), beamlet_sampler=1)
    kw = dict(n_hist=n, seed=5, n_batches=2, hist0=123)
    a = gpu_run(gctx, ph, src, **kw)
    c = G.Context(0, opts=f'{{"pass_histories": {chains - 1}}}', materials=MATS)   # one step at a time
    try:
        b = gpu_run(c, ph, src, **kw)
    finally:
        c.close()
    assert physics_events(a) == physics_events(b) and a["interactions"] == b["interactions"]
    rtol = 2 * max(sum(r["deposits"]) for r in (a, b)) * np.finfo(float).eps   # any order of all deposits
    np.testing.assert_allclose(a["dose"], b["dose"], rtol=rtol, atol=rtol * b["dose"].max())
    assert balance(a) < 1e-12
