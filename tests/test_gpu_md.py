"""GPU parity of the MD path (lj_md_*) with the oracle.

Forces, positions and velocities within 1e-10 relative over 100 FP64 steps;
fused coarse-graining counts bit-exact on the same runs (the two
trajectories differ only by the order of floating-point sums, far below the
distance of any particle to a lattice edge at these sizes); conservation
laws and determinism on the device path itself.
"""
import math

import numpy as np
import pytest

import mdlg_inputs as mi
from oracle import md as omd

pytestmark = pytest.mark.gpu


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _np(t):
    return t.detach().cpu().numpy()


def assert_moments_close(a, b, rtol=1e-13):
    """Moment sums [n, sum d^2, sum d^4, sum d_x, sum d_y] (per row) equal to
    their rounding: n exactly, the even sums relative to themselves, the odd
    ones (near zero by momentum conservation) relative to sum |d| <= sqrt(n sum d^2)."""
    a, b = np.atleast_2d(a), np.atleast_2d(b)
    assert np.array_equal(a[:, 0], b[:, 0])
    np.testing.assert_allclose(a[:, 1:3], b[:, 1:3], rtol=rtol, atol=0)
    scale = np.sqrt(np.maximum(a[:, 0] * a[:, 1], 0.0))[:, None]
    assert np.all(np.abs(a[:, 3:5] - b[:, 3:5]) <= rtol * scale)


def gpu_system(pos, vel, L, **kw):
    import paper_2101_01160_amd as m
    return m.LJSystem(_cuda(pos), _cuda(vel), box_l=L, **kw)


def oracle_advanced(n, phi, kT, seed, steps, positions="grid"):
    pos, vel, L = mi.initial_state(n, phi, kT, seed, positions)
    if steps:
        pos, vel, _, _ = omd.md_run(pos, vel, np.zeros((n, 2), np.int64), L, steps)
    return pos, vel, L


@pytest.mark.parametrize("n,phi,kT,bits", [(512, 0.0784, 20.0, 64), (2000, 0.4, 20.0, 64), (3000, 0.2, 1.0, 64),
                                           (2000, 0.4, 20.0, 32), (3000, 0.2, 1.0, 32)])
def test_forces_match_brute_force(n, phi, kT, bits):
    print(f"forces n={n} phi={phi} kT={kT} bits={bits}", flush=True)
    pos, vel, L = oracle_advanced(n, phi, kT, 7, 300)
    sysm = gpu_system(pos, vel, L, force_bits=bits)
    f = _np(sysm.forces())
    fo, _ = omd.forces(pos, L, method="brute")
    scale = np.abs(fo).max()
    tol = 1e-12 if bits == 64 else 2e-5
    assert np.max(np.abs(f - fo)) <= tol * scale
    sysm.close()


@pytest.mark.parametrize("n,phi,kT,kw", [
    (512, 0.0784, 20.0, {}),
    (512, 0.0784, 20.0, {"step_kernel": 1}),
    (2000, 0.4, 20.0, {"step_kernel": 1}),
    (1500, 0.2, 1.0, {"step_kernel": 1, "block_size": 64}),
    (1777, 0.3, 5.0, {"step_kernel": 1, "block_size": 512, "rebuild_every": 7}),
    (700, 0.4, 20.0, {"step_kernel": 1, "skin": 0.2, "rebuild_every": 3}),
    (512, 0.0784, 20.0, {"step_kernel": 2}),
    (2000, 0.4, 20.0, {"step_kernel": 2, "block_size": 128}),
    (1777, 0.3, 5.0, {"step_kernel": 2, "block_size": 64, "rebuild_every": 7}),
    (3000, 0.2, 1.0, {"step_kernel": 2, "block_size": 512}),
    (900, 0.3, 20.0, {"step_kernel": 1, "gather_batch": 16, "block_size": 128}),
    (900, 0.3, 20.0, {"step_kernel": 1, "gather_batch": 4, "block_size": 256}),
    (512, 0.0784, 20.0, {"step_kernel": 3}),
    (2000, 0.4, 20.0, {"step_kernel": 3, "block_size": 128}),
    (1777, 0.3, 5.0, {"step_kernel": 3, "block_size": 512, "rebuild_every": 7}),
    (3000, 0.2, 1.0, {"step_kernel": 3, "skin": 0.3}),
    (700, 0.4, 20.0, {"step_kernel": 3, "skin": 0.2, "rebuild_every": 3}),
])
def test_100_steps_match_oracle(n, phi, kT, kw):
    print(f"md100 n={n} phi={phi} kT={kT} {kw}", flush=True)
    pos0, vel0, L = mi.initial_state(n, phi, kT, 3)
    sysm = gpu_system(pos0, vel0, L, **kw)
    sysm.step(37)  # eager steps, then graph-replayed chunks
    sysm.step(63)
    pos, vel, img = (_np(t) for t in sysm.state())
    sysm.check()
    po, vo, io, _ = omd.md_run(pos0, vel0, np.zeros((n, 2), np.int64), L, 100)
    assert np.array_equal(img, io)
    up, uo = pos + L * img, po + L * io
    assert np.max(np.abs(up - uo)) <= 1e-10 * np.abs(uo).max()
    assert np.max(np.abs(vel - vo)) <= 1e-10 * np.abs(vo).max()
    sysm.close()


@pytest.mark.parametrize("n,nc", [(51, 3), (86, 4), (140, 5)])
def test_smallest_boxes_match_oracle(n, nc):
    """Boxes of three to five cells per side (phi = 0.4, cells of rc + skin):
    every cell's neighbourhood wraps across the periodic edges, and below
    four cells per side two cells apart are less than L / 2 apart, so the
    minimum image is taken for every pair.  100 steps against the oracle,
    with a coarse-graining event every 10 steps (counts exact)."""
    print(f"small box n={n}", flush=True)
    pos0, vel0, L = mi.initial_state(n, 0.4, 5.0, 11)
    sysm = gpu_system(pos0, vel0, L)
    assert sysm.info()["cells_per_side"] == nc
    acc = sysm.attach_cg(7, 10)
    sysm.step(100)
    pos, vel, img = (_np(t) for t in sysm.state())
    sysm.check()
    oacc = omd.CGAccum(7)
    po, vo, io, _ = omd.md_run(pos0, vel0, np.zeros((n, 2), np.int64), L, 100, cg=oacc, s_cg=10)
    assert np.array_equal(img, io)
    up, uo = pos + L * img, po + L * io
    assert np.max(np.abs(up - uo)) <= 1e-10 * np.abs(uo).max()
    assert np.max(np.abs(vel - vo)) <= 1e-10 * np.abs(vo).max()
    assert np.array_equal(_np(acc.counts)[0], oacc.counts)
    sysm.close()


def test_energy_and_momentum_match_oracle_and_are_conserved():
    n = 2000
    pos0, vel0, L = mi.initial_state(n, 0.4, 20.0, 5)
    sysm = gpu_system(pos0, vel0, L)
    e0 = sysm.energy()[0]
    o0 = omd.energy(pos0, vel0, L)
    assert e0[0] == pytest.approx(o0[0], rel=1e-13)
    assert e0[1] == pytest.approx(o0[1], rel=1e-12, abs=1e-9)
    sysm.step(2000)
    e1 = sysm.energy()[0]
    pos, vel, img = (_np(t) for t in sysm.state())
    o1 = omd.energy(pos, vel, L)
    assert e1[0] == pytest.approx(o1[0], rel=1e-12)
    assert e1[1] == pytest.approx(o1[1], rel=1e-10)
    assert abs((e1[0] + e1[1]) - (e0[0] + e0[1])) / e0[0] <= 1e-6
    assert np.max(np.abs(e1[2:] - e0[2:])) <= 1e-10 * math.sqrt(n) * math.sqrt(20.0)
    sysm.close()


def test_grid_start_potential_energy_is_zero():
    pos0, vel0, L = mi.initial_state(512, 0.0784, 20.0, 0)
    sysm = gpu_system(pos0, vel0, L)
    e = sysm.energy()[0]
    assert e[1] == 0.0
    assert e[0] == pytest.approx(511 * 20.0, rel=1e-13)
    sysm.close()


@pytest.mark.parametrize("u,kernel", [((0.0, 0.0), 1), ((0.1, -0.05), 1), ((0.0, 0.0), 2), ((0.1, -0.05), 2),
                                      ((0.0, 0.0), 3), ((0.1, -0.05), 3)])
def test_fused_coarse_graining_matches_oracle(u, kernel):
    # the CPU-sized workload: N = 512, phi = 0.0784, kT = 20, 2000 steps,
    # 32 x 32 lattice, coarse step 50 MD steps
    import torch
    n, steps, lx, s_cg = 512, 2000, 32, 50
    print(f"fused cg u={u} kernel={kernel}", flush=True)
    pos0, vel0, L = mi.initial_state(n, 0.0784, 20.0, 0)
    sysm = gpu_system(pos0, vel0, L, step_kernel=kernel)
    acc = sysm.attach_cg(lx, s_cg, u=u, cell_acc=True)
    # the fused events against the oracle's coarse-graining of the GPU's own snapshots
    ref = omd.CGAccum(lx, cell_acc=True)
    prev_p, prev_i = pos0, np.zeros((n, 2), np.int64)
    for k in range(1, steps // s_cg + 1):
        sysm.step(s_cg)
        p, _, i = (_np(t) for t in sysm.state())
        omd.coarse_grain(lx, L, prev_p, p, prev_i, i, k - 1, k, u=u, counts=ref.counts, cell_acc=ref.cell_acc,
                         moments=ref.moments)
        prev_p, prev_i = p, i.astype(np.int64)
    torch.cuda.synchronize()
    sysm.check()
    assert acc.events == steps // s_cg
    assert np.array_equal(_np(acc.counts)[0], ref.counts)
    assert np.array_equal(_np(acc.cell_acc).reshape(49, lx, lx), ref.cell_acc)
    mg = _np(acc.moments)[0]
    assert mg[0] == ref.moments[0]
    for j in range(1, 5):
        assert mg[j] == pytest.approx(ref.moments[j], rel=1e-12, abs=1e-12 * mg[1] ** 0.5)
    # and against an independent oracle run of the whole trajectory: the counts
    # agree exactly; the moments to what the chaotic growth of rounding allows
    oacc = omd.CGAccum(lx, cell_acc=True)
    omd.md_run(pos0, vel0, np.zeros((n, 2), np.int64), L, steps, cg=oacc, s_cg=s_cg, u=u)
    assert np.array_equal(_np(acc.counts)[0], oacc.counts)
    assert np.array_equal(_np(acc.cell_acc).reshape(49, lx, lx), oacc.cell_acc)
    assert mg[1] == pytest.approx(oacc.moments[1], rel=1e-6)
    assert mg[2] == pytest.approx(oacc.moments[2], rel=1e-6)
    sysm.close()


def test_coarse_step_without_divisor_near_rebuild_interval():
    """A prime coarse step (97 MD steps) keeps the rebuild interval; events then
    fall at a different offset of each graph unit.  Steps are taken one event
    at a time (graph units plus eager steps) and then five events in one call."""
    import torch
    n, lx, s_cg = 512, 32, 97
    pos0, vel0, L = mi.initial_state(n, 0.0784, 20.0, 0)
    sysm = gpu_system(pos0, vel0, L)
    K0 = sysm.info()["rebuild_every"]
    acc = sysm.attach_cg(lx, s_cg)
    K = sysm.info()["rebuild_every"]
    print(f"rebuild_every {K0} -> {K} with s_cg={s_cg}", flush=True)
    assert K == (K0 if K0 < s_cg else s_cg * (K0 // s_cg))
    for _ in range(3):
        sysm.step(s_cg)
    sysm.step(5 * s_cg)
    torch.cuda.synchronize()
    sysm.check()
    assert acc.events == 8
    oacc = omd.CGAccum(lx)
    omd.md_run(pos0, vel0, np.zeros((n, 2), np.int64), L, 8 * s_cg, cg=oacc, s_cg=s_cg)
    assert np.array_equal(_np(acc.counts)[0], oacc.counts)
    sysm.close()


@pytest.mark.parametrize("kernel", [1, 2, 3])
def test_batched_replicas_equal_single_runs(kernel):
    import torch

    import paper_2101_01160_amd as m
    print(f"batched kernel={kernel}", flush=True)
    specs = [(600, 0.0784, 20.0, 1), (1500, 0.4, 1.0, 2), (900, 0.2, 5.0, 3)]
    states = [mi.initial_state(n, phi, kT, seed) for n, phi, kT, seed in specs]
    params = [m.lj_params(s[0].shape[0], s[2], rebuild_every=10, step_kernel=kernel) for s in states]
    pos = np.concatenate([s[0] for s in states])
    vel = np.concatenate([s[1] for s in states])
    batch = m.LJSystem(_cuda(pos), _cuda(vel), params=params)
    acc = batch.attach_cg([16, 24, 20], 10)
    batch.step(60)
    bp, bv, bi = (_np(t) for t in batch.state())
    bc = _np(acc.counts)
    off = 0
    for r, (p0, v0, L) in enumerate(states):
        n = p0.shape[0]
        single = gpu_system(p0, v0, L, rebuild_every=10, step_kernel=kernel)
        sacc = single.attach_cg([16, 24, 20][r], 10)
        single.step(60)
        sp, sv, si = (_np(t) for t in single.state())
        assert np.array_equal(bp[off:off + n], sp)
        assert np.array_equal(bv[off:off + n], sv)
        assert np.array_equal(bi[off:off + n], si)
        assert np.array_equal(bc[r], _np(sacc.counts)[0])
        single.close()
        off += n
    e = batch.energy()
    assert e.shape == (3, 4)
    batch.close()
    torch.cuda.synchronize()


def test_runs_are_deterministic():
    pos0, vel0, L = mi.initial_state(3000, 0.3, 20.0, 9)
    outs = []
    for _ in range(2):
        sysm = gpu_system(pos0, vel0, L, rebuild_every=13)
        acc = sysm.attach_cg(20, 25)
        sysm.step(250)
        outs.append([_np(t) for t in sysm.state()] + [_np(acc.counts), _np(acc.moments)])
        sysm.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


def test_invalid_inputs_are_rejected():
    import paper_2101_01160_amd as m
    pos0, vel0, L = mi.initial_state(64, 0.2, 1.0, 0)
    with pytest.raises(m.MDLGError):
        gpu_system(pos0, vel0, 5.0)  # box smaller than 3 cells
    bad = pos0.copy()
    bad[3, 0] = L + 1.0
    with pytest.raises(m.MDLGError):
        gpu_system(bad, vel0, L)
    bad = vel0.copy()
    bad[5, 1] = np.nan
    with pytest.raises(m.MDLGError):
        gpu_system(pos0, bad, L)
    with pytest.raises(m.MDLGError):
        gpu_system(pos0, vel0, L, force_bits=16)
    sysm = gpu_system(pos0, vel0, L)
    with pytest.raises(m.MDLGError):
        sysm.attach_cg(4, 10)  # lattice below 7 cells
    sysm.close()


@pytest.mark.parametrize("kw", [{"step_kernel": 1}, {"step_kernel": 2}, {"step_kernel": 3},
                                {"step_kernel": 3, "skin": 0.665}])
def test_one_million_particles_sampled(kw):
    # the benchmark workload: N = 2^20 at phi = 0.0784, kT = 20, 1024^2 lattice,
    # coarse step 50, in the benchmark's launch configurations
    import torch
    n, lx, s_cg = 1 << 20, 1024, 50
    print(f"one million: init {kw}", flush=True)
    pos0, vel0, L = mi.initial_state(n, 0.0784, 20.0, 0)
    sysm = gpu_system(pos0, vel0, L, **kw)
    acc = sysm.attach_cg(lx, s_cg)
    sysm.step(s_cg)
    pos, vel, img = (_np(t) for t in sysm.state())
    f = _np(sysm.forces())
    sysm.check()
    # the coarse-graining event equals the definition on the same snapshots
    co, _, mo = omd.coarse_grain(lx, L, pos0, pos, np.zeros((n, 2), np.int64), img)
    assert np.array_equal(_np(acc.counts)[0], co)
    assert int(co.sum()) == n
    assert _np(acc.moments)[0][1] == pytest.approx(mo[1], rel=1e-10)
    # forces on the reached configuration equal the oracle's cell-list forces
    fo, _ = omd.forces(pos, L, method="cells")
    assert np.max(np.abs(f - fo)) <= 1e-12 * np.abs(fo).max()
    # one more step from the same state
    sysm.step(1)
    p1, v1, i1 = (_np(t) for t in sysm.state())
    po, vo, io, _ = omd.md_run(pos, vel, img.astype(np.int64), L, 1)
    assert np.array_equal(i1, io)
    assert np.max(np.abs((p1 + L * i1) - (po + L * io))) <= 1e-12 * L
    assert np.max(np.abs(v1 - vo)) <= 1e-12 * np.abs(vo).max()
    sysm.close()
    torch.cuda.synchronize()


def test_one_million_fused_equals_one_step():
    """The benchmark's launch configuration (three ordinary steps per launch on
    tiles of 19 cells, coarse-graining every 50 steps on the last step of a
    launch) against one step per launch on N = 2^20: the same state and
    counts bit for bit, the moments to their rounding."""
    import torch
    n, lx, s_cg = 1 << 20, 1024, 50
    pos0, vel0, L = mi.initial_state(n, 0.0784, 20.0, 0)
    out = []
    for f in (0, 1):
        print(f"one million fused={f}", flush=True)
        sysm = gpu_system(pos0, vel0, L, fuse_steps=f)
        assert sysm.info()["steps_per_launch"] == (3 if f == 0 else 1)
        acc = sysm.attach_cg(lx, s_cg)
        sysm.step(2 * s_cg + 7)
        sysm.check()
        out.append([_np(t) for t in sysm.state()] + [_np(acc.counts), _np(acc.moments)])
        sysm.close()
    for x, y in zip(out[0][:4], out[1][:4]):
        assert np.array_equal(x, y)
    assert_moments_close(out[0][4], out[1][4])
    torch.cuda.synchronize()


@pytest.mark.parametrize("kernel", [1, 2, 3])
def test_fp32_forces_track_fp64(kernel):
    # FP32 pair arithmetic: the trajectory stays within FP32 rounding of the FP64 oracle over 100 steps
    n = 2000
    print(f"fp32 kernel={kernel}", flush=True)
    pos0, vel0, L = mi.initial_state(n, 0.4, 20.0, 4)
    sysm = gpu_system(pos0, vel0, L, force_bits=32, step_kernel=kernel)
    sysm.step(100)
    pos, vel, img = (_np(t) for t in sysm.state())
    sysm.check()
    po, vo, io, _ = omd.md_run(pos0, vel0, np.zeros((n, 2), np.int64), L, 100)
    assert np.array_equal(img, io)
    assert np.max(np.abs((pos + L * img) - (po + L * io))) <= 1e-7
    assert np.max(np.abs(vel - vo)) <= 1e-4 * np.abs(vo).max()
    e = sysm.energy()[0]
    o = omd.energy(po, vo, L)
    assert e[0] + e[1] == pytest.approx(o[0] + o[1], rel=1e-6)
    sysm.close()


def test_tile_kernel_global_fallback(monkeypatch):
    # tiles whose three rows exceed the staging limit read their neighbours from
    # global memory; a limit of 0 sends every tile down that path
    monkeypatch.setenv("MDLG_TILE_STAGE_MAX", "0")
    n = 1500
    pos0, vel0, L = mi.initial_state(n, 0.3, 20.0, 8)
    sysm = gpu_system(pos0, vel0, L, step_kernel=2, block_size=128)
    acc = sysm.attach_cg(12, 20)
    sysm.step(100)
    pos, vel, img = (_np(t) for t in sysm.state())
    sysm.check()
    oacc = omd.CGAccum(12)
    po, vo, io, _ = omd.md_run(pos0, vel0, np.zeros((n, 2), np.int64), L, 100, cg=oacc, s_cg=20)
    assert np.array_equal(img, io)
    assert np.max(np.abs((pos + L * img) - (po + L * io))) <= 1e-10 * L
    assert np.array_equal(_np(acc.counts)[0], oacc.counts)
    sysm.close()


def test_autotuner_returns_runnable_params(tmp_path, monkeypatch):
    import torch

    import paper_2101_01160_amd as m
    monkeypatch.setenv("MDLG_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    specs = [(4096, 0.0784, 20.0, 1), (9000, 0.4, 1.0, 2)]
    states = [mi.initial_state(n, phi, kT, seed) for n, phi, kT, seed in specs]
    params = [m.lj_params(s[0].shape[0], s[2]) for s in states]
    pos = np.concatenate([s[0] for s in states])
    vel = np.concatenate([s[1] for s in states])
    lats = [m.Lattice(lx=20, reserved=0), m.Lattice(lx=30, reserved=0)]
    tuned, us = m.lj_md_autotune(params, _cuda(pos), _cuda(vel), 50, lats)
    assert us > 0
    assert tuned[0].step_kernel in (1, 2, 3) and tuned[0].block_size in (128, 256, 512)
    assert all(t.n == p.n and t.box_l == p.box_l for t, p in zip(tuned, params))
    # the second call is served from the cache with the same choice
    again, us2 = m.lj_md_autotune(params, _cuda(pos), _cuda(vel), 50, lats)
    assert us2 == -1.0
    assert [(t.step_kernel, t.block_size, t.skin) for t in again] == [(t.step_kernel, t.block_size, t.skin) for t in tuned]
    # the tuned launch runs and matches the oracle over 100 steps
    batch = m.LJSystem(_cuda(pos), _cuda(vel), params=tuned)
    batch.step(100)
    bp, bv, bi = (_np(t) for t in batch.state())
    batch.check()
    off = 0
    for p0, v0, L in states:
        n = p0.shape[0]
        po, vo, io, _ = omd.md_run(p0, v0, np.zeros((n, 2), np.int64), L, 100)
        assert np.array_equal(bi[off:off + n], io)
        assert np.max(np.abs((bp[off:off + n] + L * bi[off:off + n]) - (po + L * io))) <= 1e-10 * L
        off += n
    batch.close()
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,phi,kT,fuse,spl,kw", [
    (512, 0.0784, 20.0, 0, 3, {}),
    (330, 0.07, 20.0, 0, 2, {}),                  # 20 cells a side: three-step tiles too narrow
    (2000, 0.4, 20.0, 2, 2, {"block_size": 128}),
    (2000, 0.4, 20.0, 3, 3, {"block_size": 128}),
    (700, 0.4, 20.0, 2, 2, {"skin": 0.2, "rebuild_every": 3}),
    (700, 0.4, 20.0, 3, 3, {"skin": 0.2, "rebuild_every": 3}),   # ragged tiles 6, 6, 1
    (3000, 0.2, 1.0, 2, 2, {"force_bits": 32}),
    (3000, 0.2, 1.0, 3, 3, {"force_bits": 32}),
    (20000, 0.0784, 20.0, 0, 3, {"block_size": 512}),
    (20000, 0.0784, 20.0, 2, 2, {}),
])
def test_fused_steps_per_launch_equal_one(n, phi, kT, fuse, spl, kw):
    """Two or three ordinary steps per launch (tiles with a staged halo) give
    the same state and coarse-graining counts, bit for bit, as one step per
    launch, and the same displacement moments to their rounding."""
    print(f"fused n={n} phi={phi} kT={kT} fuse={fuse} {kw}", flush=True)
    pos0, vel0, L = mi.initial_state(n, phi, kT, 5)
    out = []
    for f in (fuse, 1):
        sysm = gpu_system(pos0, vel0, L, fuse_steps=f, **kw)
        assert sysm.info()["steps_per_launch"] == (spl if f != 1 else 1)
        acc = sysm.attach_cg(max(7, int(L / 2.0)), 10)
        sysm.step(13)
        sysm.step(131)
        pos, vel, img = (_np(t) for t in sysm.state())
        out.append((pos, vel, img, _np(acc.counts), _np(acc.moments)))
        sysm.close()
    for x, y in zip(out[0][:4], out[1][:4]):
        assert np.array_equal(x, y)
    # the moment partials are summed per fused tile instead of per slot tile
    assert_moments_close(out[0][4], out[1][4])


def test_paper_system_batch_fused_equals_one_step():
    """The paper-regime launch configuration: four systems of N = 99,856 in
    L = 1000 (phi = 0.0784, kT = 20) stepped as one batch, three steps per
    launch, coarse-grained on Table 1's first lattice (250^2, 3911 MD steps):
    the same states and counts, bit for bit, as one step per launch."""
    import torch

    import paper_2101_01160_amd as m
    n, L = 99856, 1000.0
    phi = n * np.pi / (4.0 * L * L)
    states = [mi.initial_state(n, phi, 20.0, 40 + r) for r in range(4)]
    pos = np.concatenate([s_[0] for s_ in states])
    vel = np.concatenate([s_[1] for s_ in states])
    out = []
    for f in (0, 1):
        print(f"paper batch fused={f}", flush=True)
        params = [m.lj_params(n, states[r][2], fuse_steps=f) for r in range(4)]
        b = m.LJSystem(_cuda(pos), _cuda(vel), params=params)
        assert b.info()["steps_per_launch"] == (3 if f == 0 else 1)
        acc = b.attach_cg([250] * 4, 391)
        b.step(2 * 391 + 5)
        b.check()
        out.append([_np(t) for t in b.state()] + [_np(acc.counts)])
        b.close()
    for x, y in zip(out[0], out[1]):
        assert np.array_equal(x, y)
    assert out[0][3].sum() == 4 * n * 2
    torch.cuda.synchronize()


def test_clustered_tile_overflow_is_reported():
    """A cluster at liquid-like density in a dilute box stages more particles
    than a three-ring tile holds: the run stops with MDLG_ECAPACITY naming the
    tile (the kernels cap what they stage and flag it)."""
    import paper_2101_01160_amd as m
    n, L, a = 2000, 200.0, 1.5
    g = np.arange(-40, 41) * a
    pts = np.stack(np.meshgrid(g, g), axis=-1).reshape(-1, 2)
    pts = pts[np.argsort((pts ** 2).sum(axis=1), kind="stable")][:n] + L / 2
    rng = np.random.default_rng(3)
    vel = rng.normal(0.0, 1.0, (n, 2))
    vel -= vel.mean(axis=0)
    print("clustered tile overflow", flush=True)
    sysm = gpu_system(pts, vel, L, fuse_steps=3)
    assert sysm.info()["steps_per_launch"] == 3
    with pytest.raises(m.MDLGError, match="tile"):
        sysm.step(10)
        sysm.check()
    sysm.close()


@pytest.mark.parametrize("fuse", [2, 3])
def test_fused_batched_replicas_equal_single(fuse):
    import paper_2101_01160_amd as m
    specs = [(4096, 0.0784, 20.0), (1500, 0.4, 1.0), (9000, 0.2, 5.0)]
    states = [mi.initial_state(n, phi, kT, 11 + i) for i, (n, phi, kT) in enumerate(specs)]
    pos = np.concatenate([s[0] for s in states])
    vel = np.concatenate([s[1] for s in states])
    params = [m.lj_params(s[0].shape[0], s[2], rebuild_every=10, fuse_steps=fuse) for s in states]
    batch = m.LJSystem(_cuda(pos), _cuda(vel), params=params)
    assert batch.info()["steps_per_launch"] == fuse
    # by default the dense replicas keep one step per launch
    dflt = m.LJSystem(_cuda(pos), _cuda(vel), params=[m.lj_params(p.n, p.box_l, rebuild_every=10) for p in params])
    assert dflt.info()["steps_per_launch"] == 1
    dflt.close()
    bacc = batch.attach_cg(12, 7)
    batch.step(55)
    bpos = _np(batch.state()[0])
    bcounts, bmom = _np(bacc.counts), _np(bacc.moments)
    batch.close()
    off = 0
    for r, (s, p) in enumerate(zip(states, params)):
        single = m.LJSystem(_cuda(s[0]), _cuda(s[1]), params=[m.lj_params(p.n, p.box_l, rebuild_every=10,
                                                                           fuse_steps=1)])
        sacc = single.attach_cg(12, 7)
        single.step(55)
        assert np.array_equal(_np(single.state()[0]), bpos[off:off + p.n])
        # coarse-graining of each replica: counts exact, moments to their rounding
        assert np.array_equal(_np(sacc.counts)[0], bcounts[r])
        assert_moments_close(bmom[r], _np(sacc.moments)[0])
        off += p.n
        single.close()


def test_save_and_resume(tmp_path):
    """lj_md_save / lj_md_load: the resumed handle starts from the saved state
    bit for bit and continues the run to within the rounding of the force sums."""
    import torch

    import paper_2101_01160_amd as m
    sizes = [1500, 700]
    states = [mi.initial_state(nr, 0.0784, 20.0, 10 + k) for k, nr in enumerate(sizes)]
    params = [m.lj_params(nr, st[2]) for nr, st in zip(sizes, states)]
    sysm = m.LJSystem(_cuda(np.concatenate([st[0] for st in states])), _cuda(np.concatenate([st[1] for st in states])),
                      params=params)
    sysm.step(300)
    p0, v0, i0 = (_np(t) for t in sysm.state())
    path = str(tmp_path / "two_replicas.state")
    sysm.save(path)
    sysm.step(100)
    pa, va, ia = (_np(t) for t in sysm.state())
    torch.cuda.synchronize()
    sysm.close()
    res = m.LJSystem.load(path)
    info = res.info()
    assert info["n_rep"] == 2 and info["n_total"] == sum(sizes) and info["steps_done"] == 300
    p1, v1, i1 = (_np(t) for t in res.state())
    assert np.array_equal(p1, p0) and np.array_equal(v1, v0) and np.array_equal(i1, i0)
    res.step(100)
    pb, vb, ib = (_np(t) for t in res.state())
    res.check()
    res.close()
    off = 0
    for nr, st in zip(sizes, states):
        L = st[2]
        sl = slice(off, off + nr)
        off += nr
        ua, ub = pa[sl] + L * ia[sl], pb[sl] + L * ib[sl]
        assert np.max(np.abs(ua - ub)) <= 1e-9 * L
        assert np.max(np.abs(va[sl] - vb[sl])) <= 1e-8 * np.max(np.abs(va[sl]))


def test_event_finish_placement_keeps_the_counts():
    """The finish of a coarse-graining event runs in the first blocks of the
    next launch, or as a kernel of its own before another event and at the
    end of every call.  Runs that end calls at events, between them and at
    whole cell-list intervals (timed graphs) give the same counts and steps;
    the moments agree to rounding (the launch plans differ).  121 fused tiles,
    more than the finish's 55 blocks, so the finish can ride on a launch."""
    import torch
    n, phi, kT, lx, s_cg = 32768, 0.0784, 20.0, 128, 50
    pos0, vel0, L = mi.initial_state(n, phi, kT, 5)
    out = []
    for mode in ("one call", "ragged calls", "timed units"):
        print(f"finish placement: {mode}", flush=True)
        sysm = gpu_system(pos0, vel0, L)
        assert sysm.info()["steps_per_launch"] == 3
        acc = sysm.attach_cg(lx, s_cg)
        if mode == "one call":
            sysm.step(1000)
        elif mode == "ragged calls":
            left = 1000
            for k in range(1000):
                c = min(left, (7, 50, 3, 43, 97)[k % 5])
                sysm.step(c)
                left -= c
                if not left:
                    break
        else:
            # the first launches, then whole intervals (the timed call aligns
            # the event phase first), then the rest
            sysm.step(50)
            K = sysm.info()["rebuild_every"]
            sysm.step_timed((1000 - 50 - K) // K, 3)  # every third interval split into timed graphs
            sysm.step(1000 - sysm.info()["steps_done"])
        torch.cuda.synchronize()
        sysm.check()
        assert sysm.info()["steps_done"] == 1000
        assert acc.events == 1000 // s_cg
        out.append((_np(acc.counts)[0].copy(), _np(acc.moments)[0].copy()))
        sysm.close()
    for c, mo in out[1:]:
        assert np.array_equal(c, out[0][0])
        assert_moments_close(mo, out[0][1])


@pytest.mark.parametrize("s_cg", [25, 50, 100])
def test_several_intervals_per_graph_equal_one_at_a_time(s_cg):
    """lj_md_step captures eight cell-list intervals to a graph where the
    coarse-step residue fixes their events (one of K and s_cg divides the
    other); the state, counts and moments equal those of calls of one
    interval each, bit for bit (the same launches in the same order)."""
    import torch
    n, phi, kT = 20000, 0.0784, 20.0
    pos0, vel0, L = mi.initial_state(n, phi, kT, 9)
    lx = int(L / 4.0)
    out = []
    for chunk in (1200, None):
        sysm = gpu_system(pos0, vel0, L, rebuild_every=50)
        acc = sysm.attach_cg(lx, s_cg)
        if chunk:
            sysm.step(chunk)
        else:
            sysm.step(2)  # the first launch and the alignment, then one interval per call
            while sysm.info()["steps_done"] + 50 <= 1200:
                sysm.step(50)
            sysm.step(1200 - sysm.info()["steps_done"])
        torch.cuda.synchronize()
        sysm.check()
        assert sysm.info()["steps_done"] == 1200 and acc.events == 1200 // s_cg
        out.append([_np(t) for t in sysm.state()] + [_np(acc.counts), _np(acc.moments)])
        sysm.close()
    for x, y in zip(out[0], out[1]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("sizes,phi,kT,kw", [
    ([40], 0.1, 20.0, {}), ([64], 0.2, 5.0, {}), ([65], 0.2, 5.0, {"rebuild_every": 1}),
    ([1023], 0.0784, 20.0, {"rebuild_every": 7}), ([1024], 0.4, 20.0, {}), ([1025], 0.3, 5.0, {"force_bits": 32}),
    ([2048], 0.0784, 20.0, {}), ([1500, 40, 700, 1999], 0.15, 10.0, {"rebuild_every": 11}),
    ([1100], 0.4, 5.0, {}), ([961 + 1024], "cluster", 0.1, {"rebuild_every": 9}),
])
def test_block_per_replica_equals_one_step(sizes, phi, kT, kw):
    """Replicas that fit one block (the default up to 2048 particles) against one step per launch: with the lists
    rebuilt at the same steps, the same states and counts bit for bit, whatever the calls; the moments to their
    rounding, and bit for bit between splits of the run."""
    import torch

    import paper_2101_01160_amd as m
    print(f"block per replica {sizes} phi={phi} {kw}", flush=True)
    if phi == "cluster":  # lists longer than LDS holds: a lattice at 1.05 beside a dilute one
        (n,), g, h = sizes, 150.0 + 1.05 * np.arange(31), 2.0 + 3.0 * np.arange(32)
        pts = np.concatenate([np.stack(np.meshgrid(x, x), axis=-1).reshape(-1, 2) for x in (g, h)])
        states = [(pts, mi.maxwell_velocities(n, kT, np.random.default_rng(2)), 300.0)]
    else:
        states = [mi.initial_state(n, phi, kT, 70 + k) for k, n in enumerate(sizes)]
    pos, vel = (np.concatenate([s[k] for s in states]) for k in (0, 1))
    out = []
    for fuse, calls in ((1, [1] * 61), (0, [61]), (0, [1, 2, 0, 17, 3, 38])):
        b = m.LJSystem(_cuda(pos), _cuda(vel), params=[m.lj_params(n, s[2], fuse_steps=fuse, **kw)
                                                       for n, s in zip(sizes, states)])
        acc = b.attach_cg([max(7, int(s[2] / 2.0)) for s in states], 5, u=(0.1, -0.3), cell_acc=True)
        for c in calls:
            b.step(c)
        b.check()
        assert acc.events == 12 and b.info()["steps_done"] == 61
        out.append([_np(t) for t in b.state()] + [_np(b.forces()), _np(acc.counts), _np(acc.cell_acc), _np(acc.moments)])
        b.close()
    for x, y, z in zip(*out):
        assert np.array_equal(y, z)
        if x is not out[0][6]:
            assert np.array_equal(x, y)
    for r in range(len(sizes)):
        assert_moments_close(out[1][6][r], out[0][6][r])
    torch.cuda.synchronize()


@pytest.mark.parametrize("sizes,phi,kT,kw", [
    ([42], 0.4, 20.0, {"block_size": 64}), ([513], 0.3, 5.0, {"block_size": 512}), ([1024], 0.4, 5.0, {"block_size": 128}),
    ([2047], 0.25, 20.0, {"rebuild_every": 6}), ([1100, 64, 1999], 0.3, 5.0, {"block_size": 64}),
    ([1025, 300], 0.4, 5.0, {"force_bits": 32, "block_size": 128}), ([1025, 300], 0.1, 5.0, {"block_size": 64}),
    ([1989], "bands", 0.1, {"block_size": 64}), ([1989], "bands", 0.1, {"block_size": 128}), ([1989], "bands", 0.1, {}),
])
def test_one_step_staged_tiles_equal_block_per_replica(sizes, phi, kT, kw):
    """The one-step list kernel at every block size against one block per replica, bit for bit: tiles of one and of
    several rows of cells, across the periodic edges, the whole box as one tile, a last tile of few particles, tiles
    whose neighbours are too many to stage (a dense band beside a dilute one), short
    lists (not staged)."""
    import paper_2101_01160_amd as m
    print(f"one step staged {sizes} phi={phi} {kw}", flush=True)
    if phi == "bands":
        L = 64.0
        g, y, x2, y2 = 0.3 + 1.05 * np.arange(60), 0.3 + 1.05 * np.arange(30), 1 + 3.0 * np.arange(21), 34 + 3.0 * np.arange(9)
        pts = np.concatenate([np.stack(np.meshgrid(a, b), axis=-1).reshape(-1, 2) for a, b in ((g, y), (x2, y2))])
        states = [(pts, mi.maxwell_velocities(sizes[0], kT, np.random.default_rng(2)), L)]
    else:
        states = [mi.initial_state(n, phi, kT, 170 + k) for k, n in enumerate(sizes)]
    pos, vel = (np.concatenate([s[k] for s in states]) for k in (0, 1))
    out = []
    for fuse in (0, 1):
        b = m.LJSystem(_cuda(pos), _cuda(vel), params=[m.lj_params(n, s[2], fuse_steps=fuse, **kw)
                                                       for n, s in zip(sizes, states)])
        acc = b.attach_cg([max(7, int(s[2] / 2.0)) for s in states], 5, u=(0.1, -0.3))
        for c in [1] * 30:  # the same rebuild steps
            b.step(c)
        b.check()
        out.append([_np(t) for t in b.state()] + [_np(acc.counts)])
        b.close()
    for x, y in zip(*out):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [900, 4096])
def test_detach_at_the_end_of_an_interval(n):
    """Detaching the coarse-graining may lengthen the interval between rebuilds.  At an interval's end a rebuild stays
    due: the particles are binned for it already (fused tiles), and there are no lists for further steps (block per
    replica)."""
    pos0, vel0, L = mi.initial_state(n, 0.0784, 20.0, 8)
    sysm = gpu_system(pos0, vel0, L)
    K0 = sysm.info()["rebuild_every"]
    s_cg = (K0 - 1) // 2
    sysm.attach_cg(20, s_cg)
    K = sysm.info()["rebuild_every"]
    assert K < K0 and K == 2 * s_cg
    sysm.step(2 * K if n <= 2048 else 2 + 2 * K)  # a fused system takes a first step and one to its alignment
    sysm.detach_cg()
    sysm.step(3)
    sysm.step(K0)
    sysm.check()
    steps = sysm.info()["steps_done"]
    pos, vel, img = (_np(t) for t in sysm.state())
    po, vo, io, _ = omd.md_run(pos0, vel0, np.zeros((n, 2), np.int64), L, steps)
    up, uo = pos + L * img, po + L * io
    # rounding grows by a factor of about ten in 100 steps of the 100-step comparisons' 1e-10
    assert np.max(np.abs(up - uo)) <= 1e-8 * np.abs(uo).max() and np.max(np.abs(vel - vo)) <= 1e-8 * np.abs(vo).max()
    sysm.close()


@pytest.mark.parametrize("sizes,phi,kT,s_cg,kw", [
    ([512], 0.0784, 20.0, 0, {"rebuild_every": 20}), ([512, 300], 0.0784, 20.0, 7, {"rebuild_every": 20}),
    ([1000], 0.35, 5.0, 0, {"rebuild_every": 25}), ([1000, 640], 0.35, 5.0, 9, {"rebuild_every": 25, "block_size": 64}),
    ([700], 0.2, 5.0, 50, {"rebuild_every": 16, "force_bits": 32}), ([1500], 0.0784, 20.0, 0, {"rebuild_every": 60}),
    ([1500, 1100], 0.0784, 20.0, 30, {"rebuild_every": 60}), ([1024], 0.0784, 20.0, 11, {"rebuild_every": 3}),
    ([1025] * 126, 0.4, 5.0, 0, {"rebuild_every": 60}), ([64], 0.1, 5.0, 0, {"rebuild_every": 30}),
])
def test_short_and_long_calls_of_small_replicas(sizes, phi, kT, s_cg, kw):
    """Long calls by one block per replica and short ones by tiles, in turn: single short calls between long ones and
    several in a row, rebuilds due in either, at their ends and between them, and tiles that have binned the particles
    for a rebuild that the other kernel finds due; events in short calls.  Against one step per launch, rebuilt at the
    same steps, the same states and counts bit for bit; moments bit for bit between two splits."""
    import paper_2101_01160_amd as m
    print(f"short and long calls {sizes[:2]} x {len(sizes)} phi={phi} s_cg={s_cg} {kw}", flush=True)
    K = kw["rebuild_every"]
    base = {n: mi.initial_state(n, phi, kT, 30 + n) for n in set(sizes)}
    pos, vel = (np.concatenate([base[n][k] for n in sizes]) for k in (0, 1))
    mixed = [1, 1, 2, K, 1, K - 1, 2 * K + 3, 1, 1, 1, 2, 3, 1, 90, 2, 2, 61, 5, 4, 1]
    mixed += [1] * (-sum(mixed) % K)                  # single steps up to the end of an interval
    mixed += [70, 1, 1, 3 * K - 72 % K, 1, 1, 1, 1, K + 1, 2, 47, 1, 46, 1, 1]
    total = sum(mixed)
    out = []
    for fuse, calls in ((1, [1] * total), (0, mixed), (0, [total]), (0, [1] * total)):
        if len(sizes) > 100 and fuse == 0 and calls is not mixed:
            continue
        b = m.LJSystem(_cuda(pos), _cuda(vel), params=[m.lj_params(n, base[n][2], fuse_steps=fuse, **kw) for n in sizes])
        acc = b.attach_cg([max(7, int(base[n][2] / 2.0)) for n in sizes], s_cg, u=(0.1, -0.3)) if s_cg else None
        for c in calls:
            b.step(c)
        b.check()
        assert b.info()["steps_done"] == total
        out.append([_np(t) for t in b.state()] + [_np(b.forces())] + ([_np(acc.counts), _np(acc.moments)] if s_cg else []))
        b.close()
    for other in out[1:]:
        for k, (x, y) in enumerate(zip(out[0], other)):
            if k == 5:
                for r in range(len(sizes)):
                    assert_moments_close(y[r], x[r])
                assert np.array_equal(y, out[1][5])
            else:
                assert np.array_equal(x, y)


def test_block_per_replica_captured_by_the_caller():
    """Steps with coarse-graining on a moving lattice, captured into a graph of the caller's and replayed with other
    work in between: the coarse step's index goes on, as if the call had been made each time."""
    import torch

    import paper_2101_01160_amd as m
    states = [mi.initial_state(n, 0.0784, 20.0, n) for n in (900, 300)]
    pos, vel = (np.concatenate([s[k] for s in states]) for k in (0, 1))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        def make():
            b = m.LJSystem(_cuda(pos), _cuda(vel), params=[m.lj_params(s[0].shape[0], s[2]) for s in states])
            return b, b.attach_cg([20, 11], 10, u=(0.37, -0.21))
        a, acc_a = make()
        b, acc_b = make()
        n = 2 * a.info()["rebuild_every"]
        a.step(n)
        b.step(n)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin()
        m.lj_md_step(a.handle, n, stream.cuda_stream)
        graph.capture_end()
        for _ in range(4):
            graph.replay()
            b.step(n)
            torch.cuda.synchronize()
            assert np.array_equal(_np(acc_a.counts), _np(acc_b.counts))
            assert np.array_equal(_np(acc_a.moments), _np(acc_b.moments))
            for x, y in zip(a.state(), b.state()):
                assert np.array_equal(_np(x), _np(y))
            assert np.array_equal(a.energy(), b.energy())
        a.check()
        b.check()
        assert _np(acc_b.counts)[0, 0] < _np(acc_b.counts)[0].sum()
        a.close()
        b.close()


def test_block_per_replica_times_the_same_parts_whatever_came_before():
    """The timed parts of an interval (ordinary steps before its first event, the rest) do not depend on the steps
    taken before the call."""
    pos0, vel0, L = mi.initial_state(900, 0.0784, 20.0, 4)
    for before in (0, 1, 13, 24, 25, 60):
        sysm = gpu_system(pos0, vel0, L)
        acc = sysm.attach_cg(20, 25)
        K = sysm.info()["rebuild_every"]
        assert K % 25 == 0
        sysm.step(before)
        ms, cnt = sysm.step_timed(9, 3)
        assert (ms > 0).all() and list(cnt) == [2 * 24, 2 * K // 25, 2]
        assert sysm.info()["steps_done"] == max(before, 1) + 9 * K and acc.events == sysm.info()["steps_done"] // 25
        sysm.check()
        sysm.close()


def test_block_per_replica_reports_drift_and_times_steps():
    pos0, vel0, L = mi.initial_state(900, 0.0784, 20.0, 4)
    sysm = gpu_system(pos0, vel0, L)
    acc = sysm.attach_cg(20, 25)
    ms, cnt = sysm.step_timed(9, 3)
    K = sysm.info()["rebuild_every"]
    assert (ms > 0).all() and sysm.info()["steps_done"] == 9 * K + 1 and cnt[2] == 2
    sysm.step(25 - (9 * K + 1) % 25)
    oacc = omd.CGAccum(20)
    steps = sysm.info()["steps_done"]
    omd.md_run(pos0, vel0, np.zeros((900, 2), np.int64), L, steps, cg=oacc, s_cg=25)
    assert acc.events == steps // 25 and np.array_equal(_np(acc.counts)[0], oacc.counts)
    sysm.check()
    sysm.close()
    import paper_2101_01160_amd as m
    sysm = gpu_system(pos0, vel0, L, rebuild_every=1000)
    with pytest.raises(m.MDLGError, match="skin"):
        sysm.step(1500)
        sysm.check()
    sysm.close()
