"""GPU parity of the displacement histograms (mdlg_displacement_hist) with the
oracle's per-pair histogram summed over every snapshot pair: bit-exact counts
on random walks (ragged batches, empty replicas, several lags and bin widths,
exact bin edges, the largest and smallest bin counts), on a trajectory of
the MD engine itself, and at the paper's system size (N = 99,856, L = 1000)."""
import math

import numpy as np
import pytest

from oracle import md as omd

pytestmark = pytest.mark.gpu


def walk(n, L, P, step, seed):
    """Random-walk snapshots wrapped into [0, L) with image counts (inputs only)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    x = rng.uniform(0.0, L, (n, 2))
    img = np.zeros((n, 2), dtype=np.int32)
    xs, imgs = [x.copy()], [img.copy()]
    for _ in range(P - 1):
        y = x + rng.normal(0.0, step, (n, 2))
        k = np.floor(y / L)
        x = y - k * L
        k[x >= L] += 1
        x[x >= L] = 0.0
        img = img + k.astype(np.int32)
        xs.append(x.copy())
        imgs.append(img.copy())
    return np.stack(xs), np.stack(imgs)


def batch(specs, P, seed=0):
    xs, imgs = [], []
    for r, (n, L, step) in enumerate(specs):
        x, i = walk(n, L, P, step, seed + r)
        xs.append(x)
        imgs.append(i)
    offsets = np.concatenate([[0], np.cumsum([s[0] for s in specs])]).astype(np.int64)
    return np.concatenate(xs, axis=1), np.concatenate(imgs, axis=1), offsets


def gpu_hist(offsets, box, xs, imgs, lags, h, n_bin, repeat=1):
    import torch

    import paper_2101_01160_amd as m
    pos = torch.from_numpy(np.ascontiguousarray(xs)).cuda()
    img = torch.from_numpy(np.ascontiguousarray(imgs, dtype=np.int32)).cuda()
    hist = torch.zeros((len(offsets) - 1, len(lags), 2, n_bin + 2), dtype=torch.int64, device="cuda")
    for _ in range(repeat):
        m.mdlg_displacement_hist(offsets, box, pos, img, lags, h, n_bin, hist)
    torch.cuda.synchronize()
    return hist.cpu().numpy()


def test_ragged_batch_matches_oracle():
    specs = [(1000, 40.0, 0.7), (0, 30.0, 0.5), (37, 25.0, 1.3), (300, 60.0, 3.0), (513, 12.0, 2.0)]
    P, lags, h, n_bin = 24, [1, 2, 5, 23], [0.05, 0.1, 0.2, 0.5], 61
    print("ragged batch", specs, lags, flush=True)
    xs, imgs, off = batch(specs, P, seed=3)
    box = [s[1] for s in specs]
    got = gpu_hist(off, box, xs, imgs, lags, h, n_bin, repeat=2)
    ref = omd.displacement_hist_series(off, box, xs, imgs, lags, h, n_bin)
    assert np.array_equal(got, 2 * ref)
    for r, (n, _, _) in enumerate(specs):
        for s, lag in enumerate(lags):
            assert (got[r, s].sum(axis=1) == 2 * n * (P - lag)).all()


@pytest.mark.parametrize("n_rep,n_bin", [(33, 24), (70, 1021)])
def test_several_launches_and_shares(n_rep, n_bin):
    """More replicas than one launch takes, ragged around whole work items, some empty; one and several histogram copies."""
    sizes = [(511, 512, 513, 0, 1, 1537)[r % 6] for r in range(n_rep)]
    xs, imgs, off = batch([(n, 10.0 + r, 0.8) for r, n in enumerate(sizes)], 5, seed=9)
    box = [10.0 + r for r in range(n_rep)]
    lags, h = [1, 3], [8.0 / n_bin, 12.0 / n_bin]
    got = gpu_hist(off, box, xs, imgs, lags, h, n_bin)
    assert np.array_equal(got, omd.displacement_hist_series(off, box, xs, imgs, lags, h, n_bin))


@pytest.mark.parametrize("n_rep,sizes", [(129, (511, 0, 513)), (513, (64, 65, 1, 0, 63)), (600, (128, 100)),
                                         (700, (257, 0, 300)), (514, (0,) * 513 + (900,))])
def test_many_replicas(n_rep, sizes):
    """One launch after another with tables as kernel arguments (to 512 replicas), one launch with tables in device
    memory (more); blocks of one to eight waves by the mean size, some replicas empty."""
    xs, imgs, off = batch([(sizes[r % len(sizes)], 10.0 + r % 7, 0.8) for r in range(n_rep)], 4, seed=n_rep)
    box = [10.0 + r % 7 for r in range(n_rep)]
    lags, h, n_bin = [1, 3], [0.3, 0.5], 24
    got = gpu_hist(off, box, xs, imgs, lags, h, n_bin)
    assert np.array_equal(got, omd.displacement_hist_series(off, box, xs, imgs, lags, h, n_bin))


@pytest.mark.parametrize("n_bin", [1, 2, 4094])
def test_bin_count_extremes(n_bin):
    specs = [(700, 20.0, 1.0), (129, 33.0, 0.4)]
    P, lags = 9, [1, 8]
    h = [4.0 / n_bin, 9.0 / n_bin]
    print("n_bin", n_bin, flush=True)
    xs, imgs, off = batch(specs, P, seed=17)
    box = [s[1] for s in specs]
    got = gpu_hist(off, box, xs, imgs, lags, h, n_bin)
    ref = omd.displacement_hist_series(off, box, xs, imgs, lags, h, n_bin)
    assert np.array_equal(got, ref)


def test_exact_edges_and_far_displacements():
    """Dyadic displacements that land exactly on bin edges, beyond the range
    on either side, and across many periodic images."""
    rng = np.random.default_rng(2)
    n, L, P = 500, 16.0, 3
    x0 = np.floor(rng.uniform(0, L, (n, 2)) * 16) / 16
    d = rng.integers(-40, 41, (P - 1, n, 2)) * 0.25
    d[0, :5] = [[1e3, -1e3], [-1e3, 1e3], [4.0, -4.0], [-4.0, 4.0], [3.75, -3.75]]
    xs, imgs = [x0], [np.zeros((n, 2), np.int64)]
    u = x0.copy()
    for p in range(P - 1):
        u = u + d[p]
        k = np.floor(u / L).astype(np.int64)
        xs.append(u - L * k)
        imgs.append(k)
    xs = np.stack(xs)
    imgs = np.stack(imgs).astype(np.int32)
    off = np.array([0, n], dtype=np.int64)
    got = gpu_hist(off, [L], xs, imgs, [1, 2], [0.25, 0.5], 32)
    ref = omd.displacement_hist_series(off, [L], xs, imgs, [1, 2], [0.25, 0.5], 32)
    assert np.array_equal(got, ref)
    assert got[0, 0, :, 32].sum() > 0 and got[0, 0, :, 33].sum() > 0


def test_md_trajectory_matches_oracle():
    """Snapshots of the GPU MD engine (phi = 0.0784, kT = 20) every 50 steps."""
    import torch

    import mdlg_inputs as mi
    import paper_2101_01160_amd as m
    n, P = 4096, 12
    pos0, vel0, L = mi.initial_state(n, 0.0784, 20.0, seed=5)
    sysm = m.LJSystem(torch.from_numpy(pos0).cuda(), torch.from_numpy(vel0).cuda(), box_l=L)
    xs, imgs = [], []
    for p in range(P):
        if p:
            sysm.step(50)
        x, _, i = sysm.state()
        xs.append(x.cpu().numpy())
        imgs.append(i.cpu().numpy())
    sysm.close()
    xs, imgs = np.stack(xs), np.stack(imgs)
    off = np.array([0, n], dtype=np.int64)
    lags = [1, 4, 11]
    sd = [math.sqrt(2 * 20.0) * 50e-4 * l for l in lags]   # ballistic scale v_th t
    h = [s / 10 for s in sd]
    got = gpu_hist(off, [L], xs, imgs, lags, h, 121)
    ref = omd.displacement_hist_series(off, [L], xs, imgs, lags, h, 121)
    assert np.array_equal(got, ref)
    assert got[0, 0, :, 121:].sum() < 1e-3 * got[0, 0].sum()


def test_paper_size_matches_oracle():
    """N = 99,856 in L = 1000 (the paper's system), 17 snapshots, 3 lags."""
    n, L, P = 99856, 1000.0, 17
    lags, h, n_bin = [1, 4, 16], [0.05, 0.1, 0.2], 201
    print("paper size", n, P, flush=True)
    xs, imgs, off = batch([(n, L, 1.2)], P, seed=9)
    got = gpu_hist(off, [L], xs, imgs, lags, h, n_bin)
    ref = omd.displacement_hist_series(off, [L], xs, imgs, lags, h, n_bin)
    assert np.array_equal(got, ref)


def test_invalid_arguments_raise():
    import torch

    import paper_2101_01160_amd as m
    xs, imgs, off = batch([(64, 10.0, 0.5)], 4)
    pos = torch.from_numpy(xs).cuda()
    img = torch.from_numpy(imgs).cuda()

    def call(lags=(1,), h=(0.1,), n_bin=8, box=(10.0,), offsets=off):
        hist = torch.zeros((1, len(lags), 2, max(n_bin, 0) + 2), dtype=torch.int64, device="cuda")
        m.mdlg_displacement_hist(offsets, box, pos, img, list(lags), list(h), n_bin, hist)

    call()
    for kw in (dict(lags=(4,)), dict(lags=(0,)), dict(h=(0.0,)), dict(h=(float("nan"),)), dict(n_bin=0),
               dict(n_bin=4095), dict(box=(-1.0,)), dict(lags=tuple(range(1, 66)), h=(0.1,) * 65)):
        with pytest.raises(m.MDLGError):
            call(**kw)
