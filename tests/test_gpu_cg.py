"""GPU parity of the standalone coarse-graining (mdlg_coarse_grain) with the
oracle: integer outputs bit-exact, moments within 1e-12 relative."""
import math

import numpy as np
import pytest

from oracle import md as omd
from tests import _sources as src

pytestmark = pytest.mark.gpu


def _cuda(a, dtype=None):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda()


def run_gpu(lx, L, x0, x1, i0, i1, k0=0, k1=1, u=(0.0, 0.0), dense=True, acc=True):
    import torch

    import paper_2101_01160_amd as m
    n = x0.shape[0]
    counts = torch.zeros(50, dtype=torch.int64, device="cuda")
    moments = torch.zeros(5, dtype=torch.float64, device="cuda")
    n_event = torch.full((49, lx, lx), 7, dtype=torch.int32, device="cuda") if dense else None
    cell_acc = torch.zeros((49, lx, lx), dtype=torch.int32, device="cuda") if acc else None
    ip = None if i0 is None else _cuda(i0, torch.int32)
    ic = None if i1 is None else _cuda(i1, torch.int32)
    m.mdlg_coarse_grain(lx, L, _cuda(x0), _cuda(x1), counts, moments, ip, ic, k0, k1, u, n_event, cell_acc)
    torch.cuda.synchronize()
    return (counts.cpu().numpy(), None if n_event is None else n_event.cpu().numpy(), moments.cpu().numpy(),
            None if cell_acc is None else cell_acc.cpu().numpy())


def compare(lx, L, x0, x1, i0, i1, k0=0, k1=1, u=(0.0, 0.0)):
    print(f"coarse_grain n={x0.shape[0]} lx={lx} L={L:.3f} k=({k0},{k1}) u={u}", flush=True)
    cg, ng, mg, ag = run_gpu(lx, L, x0, x1, i0, i1, k0, k1, u)
    co, no, mo = omd.coarse_grain(lx, L, x0, x1, i0, i1, k0, k1, u=u, dense=True)
    assert np.array_equal(cg, co)
    assert np.array_equal(ng, no)
    assert np.array_equal(ag, no)
    assert mg[0] == mo[0]
    for j in range(1, 5):
        assert mg[j] == pytest.approx(mo[j], rel=1e-12, abs=1e-12 * math.sqrt(max(mo[1], 1e-300)))
    return cg


@pytest.mark.parametrize("n", [1, 63, 256, 1000, 4097, 100_003])
def test_gaussian_steps_ragged_sizes(n):
    rng = np.random.default_rng(n)
    lx, L = 32, 71.618
    x0, x1, i0, i1 = src.gaussian_step(rng, n, L, var=(1.2 * L / lx) ** 2)
    compare(lx, L, x0, x1, i0, i1)


def test_integer_displacements_and_overflow():
    rng = np.random.default_rng(1)
    lx, L, n = 64, 140.0, 200_000
    x0, x1, i0, i1, v = src.integer_step(rng, n, lx, L, vmax=5)
    c = compare(lx, L, x0, x1, i0, i1)
    assert c[49] > 0 and c.sum() == n


@pytest.mark.parametrize("n,shift,k", [(3 * 1024 * 256 + 1, 0, 0), (5 * 1024 * 256 + 77, 0, 0), (5000, 1001, 0),
                                       (5000, 100_000_000, 0), (5000, 0, 700_000_000), (5000, 0, -700_000_000)])
def test_block_limit_and_wide_coordinates(n, shift, k):
    """More particles than one pass of the most blocks takes; image differences and lattice coordinates on either side
    of what the 32-bit path holds (particles that stay, and some whose images differ by `shift`)."""
    rng = np.random.default_rng(n)
    lx, L = 20, 40.0
    x0, x1, i0, i1 = src.gaussian_step(rng, n, L, var=(0.8 * L / lx) ** 2)
    i1 = i1 + shift * (np.arange(n)[:, None] % 7 == 0)
    compare(lx, L, x0, x1, i0, i1, k0=k, k1=k + 1, u=(0.25, -0.125) if k else (0.0, 0.0))


@pytest.mark.parametrize("noalloc", [False, True])
def test_image_counts_at_the_ends_of_their_range(noalloc):
    """Image counts whose difference leaves 32 bits are an overflow event, also where a particle crosses the box edge and
    what 32 bits leave of the difference is that crossing; with the same large images at both ends particles move as
    ever."""
    import torch

    import paper_2101_01160_amd as m
    n, lx, L = 3000, 20, 40.0
    rng = np.random.default_rng(5)
    x0, x1, i0, i1 = src.gaussian_step(rng, n, L, var=(0.8 * L / lx) ** 2)
    lo, hi = -2**31, 2**31 - 1
    i0, i1 = i0.copy(), i1.copy()
    x0[0::9], x1[0::9] = rng.uniform(L - 2.0, L, x0[0::9].shape), rng.uniform(0.0, 2.0, x0[0::9].shape)
    x0[1::9], x1[1::9] = rng.uniform(0.0, 2.0, x0[1::9].shape), rng.uniform(L - 2.0, L, x0[1::9].shape)
    for k, (a, b) in enumerate(((hi, lo), (lo, hi), (hi - 500, lo + 400), (lo + 3, hi - 7), (hi, hi), (lo, lo))):
        i0[k::9], i1[k::9] = a, b
    counts = torch.zeros(50, dtype=torch.int64, device="cuda")
    acc = torch.zeros((49, lx, lx), dtype=torch.int32, device="cuda")
    m.mdlg_coarse_grain(lx, L, _cuda(x0), _cuda(x1), counts, None, _cuda(i0, torch.int32), _cuda(i1, torch.int32),
                        cell_acc=acc, noalloc=noalloc)
    torch.cuda.synchronize()
    co, no, _ = omd.coarse_grain(lx, L, x0, x1, i0, i1, dense=True)
    assert np.array_equal(counts.cpu().numpy(), co) and np.array_equal(acc.cpu().numpy(), no)
    assert co[49] >= 4 * (n // 9)


def test_images_and_frame_shift():
    rng = np.random.default_rng(2)
    lx, L, n = 50, 100.0, 50_000
    x0, x1, i0, i1 = src.wsg_step(rng, n, L, mu2=(0.7 * L / lx) ** 2, lam=1.2)
    # both snapshots carry image counts
    i0 = rng.integers(-3, 4, (n, 2)).astype(np.int64)
    i1 = i1 + i0
    compare(lx, L, x0, x1, i0, i1, k0=17, k1=18, u=(0.13, -0.19))
    compare(lx, L, x0, x1, i0, i1, k0=1000, k1=1001, u=(-0.2, 0.05))


def test_null_images_and_empty_input():
    import torch

    import paper_2101_01160_amd as m
    rng = np.random.default_rng(3)
    lx, L, n = 16, 30.0, 3000
    x0 = rng.uniform(0, L, (n, 2))
    x1 = np.mod(x0 + rng.normal(0, 0.5, (n, 2)), L)
    compare(lx, L, x0, x1, None, None)
    counts = torch.zeros(50, dtype=torch.int64, device="cuda")
    e = torch.empty((0, 2), dtype=torch.float64, device="cuda")
    m.mdlg_coarse_grain(lx, L, e, e, counts)
    torch.cuda.synchronize()
    assert int(counts.sum()) == 0


def test_counts_accumulate_and_cell_boundaries():
    # positions exactly on cell edges: the floor rule puts them in the upper cell
    lx, L = 10, 25.0
    dxl = L / lx
    g = np.arange(lx) * dxl
    x0 = np.stack(np.meshgrid(g, g), axis=-1).reshape(-1, 2)
    x1 = x0.copy()
    x1[:, 0] = np.mod(x1[:, 0] + dxl, L)
    i1 = np.zeros_like(x0, dtype=np.int64)
    i1[:, 0] = (x0[:, 0] + dxl >= L).astype(np.int64)
    c = compare(lx, L, x0, x1, np.zeros_like(i1), i1)
    assert c[1] == lx * lx


def test_large_lattice_one_million():
    rng = np.random.default_rng(4)
    lx, L, n = 1024, 3241.058, 1 << 20
    x0, x1, i0, i1 = src.gaussian_step(rng, n, L, var=0.02)
    compare(lx, L, x0, x1, i0, i1)


def test_invalid_arguments_are_rejected():
    import torch

    import paper_2101_01160_amd as m
    x = torch.zeros((4, 2), dtype=torch.float64, device="cuda")
    counts = torch.zeros(50, dtype=torch.int64, device="cuda")
    with pytest.raises(m.MDLGError):
        m.mdlg_coarse_grain(0, 10.0, x, x, counts)
    with pytest.raises(m.MDLGError):
        m.mdlg_coarse_grain(8, -1.0, x, x, counts)
    with pytest.raises(ValueError):
        m.mdlg_coarse_grain(8, 10.0, x.float(), x, counts)
