"""C-ABI library: loads, exports every declared symbol, and its host FP64 code
(equilibria, lambda, measured f_eq) matches the oracle.  No GPU is touched."""
import os
import re

import numpy as np
import pytest

from oracle import closed_forms as cf
from oracle import lattice

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    txt = open(os.path.join(ROOT, "include", "mdlg.h")).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b((?:lj_md|mdlg)_\w+)\s*\(", txt)))


def test_library_exports_every_declared_symbol():
    import ctypes

    from paper_2101_01160_amd import _abi
    lib = ctypes.CDLL(_abi.LIBPATH)
    names = declared_functions()
    assert len(names) >= 20
    for name in names:
        assert hasattr(lib, name), name
    assert sorted(_abi.EXPORTS) == names


def test_velocity_table_matches_oracle_numbering():
    import paper_2101_01160_amd as m
    assert np.array_equal(m.mdlg_velocity_table(), lattice.d2q49())


CASES = [(1e-4, (0.0, 0.0)), (0.02, (0.0, 0.0)), (0.1611, (0.0, 0.0)), (1 / 6, (0.0, 0.0)),
         (0.1611, (0.13, -0.07)), (0.4, (0.2, 0.1)), (0.05, (-0.2, 0.19))]


@pytest.mark.parametrize("a2,u", CASES)
def test_gauss_matches_oracle(a2, u):
    import paper_2101_01160_amd as m
    assert np.max(np.abs(m.mdlg_feq_gauss(a2, u) - cf.feq_gauss(a2, u))) <= 1e-14


@pytest.mark.parametrize("a2,u", CASES[::2])
@pytest.mark.parametrize("lam", [0.1, 1.3, 6.0, 40.0])
def test_wsg_matches_oracle(a2, u, lam):
    import paper_2101_01160_amd as m
    assert np.max(np.abs(m.mdlg_feq_wsg(a2, lam, u) - cf.feq_wsg(a2, lam, u))) <= 1e-14


def test_wsg_zero_lambda_is_gauss():
    import paper_2101_01160_amd as m
    assert np.array_equal(m.mdlg_feq_wsg(0.1611, 0.0), m.mdlg_feq_gauss(0.1611))


@pytest.mark.parametrize("lam", [0.01, 0.3, 0.8, 1.7, 12.0, 300.0])
def test_lambda_matches_printed_roots(lam):
    import paper_2101_01160_amd as m
    mu2 = 3.3
    mu4 = cf.wsg_mu4(mu2, lam)
    l1, l2 = cf.lambda_roots(mu2, mu4)
    got2, r = m.mdlg_lambda_from_moments(mu2, mu4, 2)
    got1, _ = m.mdlg_lambda_from_moments(mu2, mu4, 1)
    assert got2 == pytest.approx(l2, rel=1e-9)
    assert got1 == pytest.approx(l1, rel=1e-9)
    assert r == pytest.approx(mu4 / (3 * mu2 ** 2), rel=1e-15)


def test_lambda_edge_readings_match_oracle():
    import paper_2101_01160_amd as m
    for mu4 in [2.0, 3.0, 3.75, 4.5]:
        assert m.mdlg_lambda_from_moments(1.0, mu4)[0] == cf.lambda_from_moments(1.0, mu4)[0]


def test_measured_matches_oracle():
    import paper_2101_01160_amd as m
    rng = np.random.default_rng(3)
    counts = rng.integers(0, 10 ** 9, 50).astype(np.int64)
    for sym in (False, True):
        g, ovf = m.mdlg_feq_measured(counts, 123457, 40, sym)
        go, ovo = cf.feq_measured(counts, 123457, 40)
        if sym:
            go = cf.symmetrize(go)
        assert np.max(np.abs(g - go) / go) <= 1e-15
        assert ovf == ovo


def test_moments_helper():
    import paper_2101_01160_amd as m
    mu2, mu4, a2 = m.mdlg_moments([10.0, 5.0, 7.5, 0.0, 0.0], 2.0)
    assert (mu2, mu4, a2) == (0.5, 0.75, 0.125)


def test_invalid_arguments_raise():
    import paper_2101_01160_amd as m
    with pytest.raises(m.MDLGError):
        m.mdlg_feq_gauss(-1.0)
    with pytest.raises(m.MDLGError):
        m.mdlg_feq_wsg(0.1, -2.0)
    with pytest.raises(m.MDLGError):
        m.mdlg_lambda_from_moments(0.0, 1.0)
    with pytest.raises(m.MDLGError):
        m.mdlg_feq_measured(np.zeros(50, np.int64), 0, 1)


@pytest.mark.parametrize("msd,lam,mean,h,n_bin", [(1.0, 0.0, 0.0, 0.25, 41), (0.0123, 0.7, 0.003, 0.02, 31),
                                                  (2.5, 3.0, -0.4, 0.3, 60), (1e-3, 12.0, 0.0, 0.01, 17),
                                                  (4.0, 0.2, 1.0, 0.05, 1)])
def test_pdf_bins_match_oracle(msd, lam, mean, h, n_bin):
    import paper_2101_01160_amd as m
    pg, pw = m.mdlg_pdf_bins(msd, lam, mean, h, n_bin)
    rg, rw = cf.pdf_bins(msd, lam, mean, h, n_bin)
    for got, ref in ((pg, rg), (pw, rw)):
        assert np.allclose(got, ref, rtol=1e-12, atol=1e-16)
    assert pg.sum() == pytest.approx(1.0, abs=1e-14) and pw.sum() == pytest.approx(1.0, abs=1e-14)


def test_pdf_measured_and_kl_match_oracle():
    import paper_2101_01160_amd as m
    rng = np.random.default_rng(6)
    hist = rng.integers(0, 1000, (2, 3, 2, 45)).astype(np.int64)
    hist[..., 7] = 0
    assert np.allclose(m.mdlg_pdf_measured(hist), cf.pdf_measured(hist), rtol=1e-15, atol=0)
    r = cf.pdf_measured(hist)
    q = cf.pdf_bins(0.8, 1.5, 0.0, 0.1, 43)[1]
    k, d = m.mdlg_kl_divergence(r, q)
    assert np.allclose(k, cf.kl_elementwise(r, q), rtol=1e-13, atol=1e-300)
    assert k[7] == 0.0
    assert d == pytest.approx(cf.kl_divergence(r, q), rel=1e-13)
    k, d = m.mdlg_kl_divergence(q, q)
    assert d == 0.0 and not k.any()
    k, d = m.mdlg_kl_divergence([0.5, 0.5], [1.0, 0.0])
    assert np.isinf(d) and np.isinf(k[1]) and k[0] == pytest.approx(0.5 * np.log(0.5))


def test_pdf_invalid_arguments_raise():
    import paper_2101_01160_amd as m
    for args in ((0.0, 1.0, 0.0, 0.1, 10), (1.0, -1.0, 0.0, 0.1, 10), (1.0, 1.0, 0.0, 0.0, 10),
                 (1.0, 1.0, 0.0, 0.1, 0), (1.0, 1.0, 0.0, 0.1, 4095), (1.0, 1.0, np.inf, 0.1, 10)):
        with pytest.raises(m.MDLGError):
            m.mdlg_pdf_bins(*args)
    with pytest.raises(m.MDLGError):
        m.mdlg_pdf_measured(np.zeros((2, 5), np.int64))
    with pytest.raises(m.MDLGError):
        m.mdlg_pdf_measured(np.array([1, -1, 3]))
    with pytest.raises(m.MDLGError):
        m.mdlg_kl_divergence([0.5, np.nan], [0.5, 0.5])
    with pytest.raises(m.MDLGError):
        m.mdlg_kl_divergence([0.5, 0.5], [-0.5, 1.5])


def test_lambda_vacf_matches_oracle():
    import paper_2101_01160_amd as m
    rng = np.random.default_rng(9)
    t = np.concatenate([[0.0], np.cumsum(rng.uniform(0.01, 0.05, 199))])
    for c in (40.0 * np.exp(-t / 0.6) + rng.normal(0, 0.05, t.size), np.full(t.size, 2.0)):
        c[0] = abs(c[0]) + 1.0
        for cut in (0.01, 0.1):
            got = m.mdlg_lambda_vacf(t, c, 0.3911, cut)
            ref = cf.lambda_vacf(t, c, 0.3911, cut)
            assert got == pytest.approx(ref, rel=1e-13)
    for bad in ((t, -c, 1.0), (t[::-1].copy(), c, 1.0), (t, c, 0.0)):
        with pytest.raises(m.MDLGError):
            m.mdlg_lambda_vacf(*bad)


def test_state_load_rejects_missing_and_foreign_files(tmp_path):
    """The file is read and checked before any device call (stream NULL)."""
    import ctypes

    from paper_2101_01160_amd import _abi
    bad = tmp_path / "foreign.state"
    bad.write_bytes(b"not a state file" * 8)
    for path in (tmp_path / "missing.state", bad):
        h = ctypes.c_void_p()
        assert _abi.lib().lj_md_load(ctypes.byref(h), str(path).encode(), None) == -1  # MDLG_EINVAL
        assert not h.value
        assert b"lj_md_load" in _abi.lib().mdlg_last_error()


@pytest.mark.parametrize("n_snap,n_lag", [(100, 20), (20, 3), (20000, 3)])
@pytest.mark.parametrize("sizes", [[2**32], [2**31, 2**31 - 300, 300], [1] + [2**32 - 256]])
def test_vacf_refuses_the_same_sizes_on_every_route(n_snap, n_lag, sizes):
    """2^24 blocks of 256 particles or more are refused before anything touches the device, also where the trajectories
    would be staged in LDS."""
    import ctypes as C

    from paper_2101_01160_amd import _abi
    off = (C.c_int64 * (len(sizes) + 1))(0, *np.cumsum(sizes).tolist())
    lags = (C.c_int32 * n_lag)(*range(n_lag))
    host = (C.c_double * 4)()
    rc = _abi.lib().mdlg_vacf(len(sizes), off, n_snap, C.cast(host, C.c_void_p), n_lag, lags, C.cast(host, C.c_void_p), None)
    assert rc == -1 and b"too many particles" in _abi.lib().mdlg_last_error()


def test_noalloc_states_its_limit_as_the_calls_own():
    """The limit is the interface's: the scratch of a call does not grow with the number of particles."""
    import ctypes as C

    from paper_2101_01160_amd import _abi
    lat = _abi.Lattice(lx=8, reserved=0, u=(C.c_double * 2)(0.0, 0.0))
    host = (C.c_double * 4)()
    p = C.cast(host, C.c_void_p)
    rc = _abi.lib().mdlg_coarse_grain_noalloc(C.byref(lat), 10.0, _abi.NOALLOC_MAX_N + 1, p, None, 0, p, None, 1, p, None,
                                              None, None, None)
    msg = _abi.lib().mdlg_last_error().decode()
    assert rc == -1 and str(_abi.NOALLOC_MAX_N) in msg and "scratch" not in msg
