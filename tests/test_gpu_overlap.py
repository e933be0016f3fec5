"""GPU parity of the projection, the polynomial sign and the overlap operator."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import dense, dirac, sign
from oracle.lattice import Lattice

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1106_4964_amd import ovl  # noqa: E402

import gpu_util as gu  # noqa: E402

RHO = 1.5


def _lowmodes_dev(g, V):
    dev = gu.pack(g, V.reshape(len(V), g.N, 4, 3), ovl.OVL_F64, len(V))
    return dev


@pytest.fixture(scope="module")
def c1():
    """4^4, c = 0.3, seeds 1/101, exact spectral bounds from the dense H_w."""
    dims = (4, 4, 4, 4)
    lat = Lattice(dims)
    U = si.gauge_field(dims, 0.3, 1)
    H = dense.dense_hw(lat, U, RHO)
    w = np.linalg.eigvalsh(H)
    return dict(dims=dims, lat=lat, U=U, lo=float(np.min(np.abs(w))), hi=float(np.max(np.abs(w))),
                psi=si.gaussian_spinor(dims, 101))


def test_sign_c1_degree200_f64(c1):
    """4^4 config: polynomial of degree 200, no projection, FP64 to 1e-12."""
    g = ovl.Geometry(c1["dims"])
    gauge = gu.make_gauge(g, c1["U"])
    s_lib = ovl.Sign(c1["lo"], c1["hi"], n=200)
    s_or = sign.make_sign(c1["lo"], c1["hi"], 200)
    inp = gu.pack(g, c1["psi"], ovl.OVL_F64)
    out = gu.empty_field(g, ovl.OVL_F64)
    ovl.ovl_sign_apply(out, inp, gauge, RHO, s_lib, None, ovl.OVL_F64, 1, None)
    got = gu.unpack(g, out, ovl.OVL_F64)
    want = sign.sign_apply(c1["lat"], c1["U"], c1["psi"], RHO, s_or)
    assert gu.max_rel_err(got, want) < 1e-12


@pytest.mark.parametrize("dagger", [0, 1])
@pytest.mark.parametrize("m", [0.01, 0.05])
def test_overlap_c1_f64(c1, dagger, m):
    g = ovl.Geometry(c1["dims"])
    gauge = gu.make_gauge(g, c1["U"])
    s_lib = ovl.Sign(c1["lo"], c1["hi"], n=200)
    s_or = sign.make_sign(c1["lo"], c1["hi"], 200)
    inp = gu.pack(g, c1["psi"], ovl.OVL_F64)
    out = gu.empty_field(g, ovl.OVL_F64)
    ovl.ovl_overlap_apply(out, inp, gauge, RHO, m, s_lib, None, dagger, ovl.OVL_F64, 1, None)
    got = gu.unpack(g, out, ovl.OVL_F64)
    want = sign.overlap_apply(c1["lat"], c1["U"], c1["psi"], RHO, m, s_or, dagger=bool(dagger))
    assert gu.max_rel_err(got, want) < 1e-12


@pytest.mark.parametrize("nrhs", [1, 3, 12])
def test_projection_parity(nrhs):
    dims = (6, 6, 6, 8)
    g = ovl.Geometry(dims)
    ell = 21
    V = si.orthonormal_spinors(dims, ell, seed=7)
    lam = np.linspace(-0.9, 0.8, ell)
    lm = ovl.LowModes(g, _lowmodes_dev(g, V), lam)
    psi = np.stack([si.gaussian_spinor(dims, 30 + r) for r in range(nrhs)])
    inp = gu.pack(g, psi, ovl.OVL_F64, nrhs)
    ph = gu.empty_field(g, ovl.OVL_F64, nrhs)
    w = gu.empty_field(g, ovl.OVL_F64, nrhs)
    ovl.ovl_lowmodes_project(lm, inp, ph, w, ovl.OVL_F64, nrhs, None)
    got_h = gu.unpack(g, ph, ovl.OVL_F64, nrhs).reshape(nrhs, g.N, 4, 3)
    got_w = gu.unpack(g, w, ovl.OVL_F64, nrhs).reshape(nrhs, g.N, 4, 3)
    for r in range(nrhs):
        c, want_h = sign.project_low(V, psi[r])
        want_w = ((np.sign(lam) * c) @ V.reshape(ell, -1)).reshape(g.N, 4, 3)
        assert gu.max_rel_err(got_h[r], want_h) < 1e-13
        assert gu.max_rel_err(got_w[r], want_w) < 1e-13


@pytest.mark.parametrize("nrhs", [1, 12])
@pytest.mark.parametrize("prec", [ovl.OVL_F32, ovl.OVL_F16, ovl.OVL_BF16])
def test_projection_parity_low_precision(prec, nrhs):
    """Batches below FP64 (FP64 basis, FP64 accumulation): psi_h and w
    against the oracle's FP64 projection of the same stored input, element
    by element, to the output precision's rounding."""
    dims = (6, 6, 6, 8)
    g = ovl.Geometry(dims)
    ell = 21
    V = si.orthonormal_spinors(dims, ell, seed=7)
    lam = np.linspace(-0.9, 0.8, ell)
    lm = ovl.LowModes(g, _lowmodes_dev(g, V), lam)
    psi = np.stack([si.gaussian_spinor(dims, 30 + r) for r in range(nrhs)])
    inp = gu.pack(g, psi, prec, nrhs)
    psi_stored = gu.unpack(g, inp, prec, nrhs).reshape(nrhs, g.N, 4, 3)
    ph = gu.empty_field(g, prec, nrhs)
    w = gu.empty_field(g, prec, nrhs)
    ovl.ovl_lowmodes_project(lm, inp, ph, w, prec, nrhs, None)
    got_h = gu.unpack(g, ph, prec, nrhs).reshape(nrhs, g.N, 4, 3)
    got_w = gu.unpack(g, w, prec, nrhs).reshape(nrhs, g.N, 4, 3)
    bound = 4 * gu.UNIT_ROUNDOFF[prec] + 1e-12
    worst = 0.0
    for r in range(nrhs):
        c, want_h = sign.project_low(V, psi_stored[r])
        want_w = ((np.sign(lam) * c) @ V.reshape(ell, -1)).reshape(g.N, 4, 3)
        worst = max(worst, gu.max_rel_err(got_h[r], want_h), gu.max_rel_err(got_w[r], want_w))
    print("projection, precision %d, %d rhs: max rel err %.2e (bound %.2e)" % (prec, nrhs, worst, bound))
    assert worst < bound


@pytest.mark.parametrize("dagger", [0, 1])
def test_overlap_with_lowmodes_f64_ragged(dagger):
    """6x6x6x8 (ragged tiles), synthetic orthonormal 'low modes', 12 RHS."""
    dims = (6, 6, 6, 8)
    lat = Lattice(dims)
    g = ovl.Geometry(dims)
    U = si.gauge_field(dims, 0.25, 2)
    gauge = gu.make_gauge(g, U)
    ell = 9
    V = si.orthonormal_spinors(dims, ell, seed=3)
    lam = np.array([0.3, -0.31, 0.35, -0.4, 0.41, 0.45, -0.5, 0.52, -0.55])
    lm = ovl.LowModes(g, _lowmodes_dev(g, V), lam)
    s_lib = ovl.Sign(0.55, 6.6, n=40)
    s_or = sign.make_sign(0.55, 6.6, 40)
    nrhs = 12
    psi = np.stack([si.gaussian_spinor(dims, 50 + r) for r in range(nrhs)])
    inp = gu.pack(g, psi, ovl.OVL_F64, nrhs)
    out = gu.empty_field(g, ovl.OVL_F64, nrhs)
    ovl.ovl_overlap_apply(out, inp, gauge, RHO, 0.01, s_lib, lm, dagger, ovl.OVL_F64, nrhs, None)
    got = gu.unpack(g, out, ovl.OVL_F64, nrhs)
    for r in (0, 5, 11):
        want = sign.overlap_apply(lat, U, psi[r], RHO, 0.01, s_or, V, lam, dagger=bool(dagger))
        assert gu.max_rel_err(got[r], want) < 1e-12


@pytest.mark.parametrize("prec", [ovl.OVL_F32, ovl.OVL_F16, ovl.OVL_BF16])
def test_overlap_low_precision_error(c1, prec):
    """Error of the low-precision overlap apply against the FP64 oracle (stated)."""
    g = ovl.Geometry(c1["dims"])
    gauge = gu.make_gauge(g, c1["U"], [(prec, 1)])
    n = 120
    s_lib = ovl.Sign(c1["lo"], c1["hi"], n=n)
    s_or = sign.make_sign(c1["lo"], c1["hi"], n)
    inp = gu.pack(g, c1["psi"], prec)
    out = gu.empty_field(g, prec)
    ovl.ovl_overlap_apply(out, inp, gauge, RHO, 0.01, s_lib, None, 0, prec, 1, None)
    got = gu.unpack(g, out, prec)
    want = sign.overlap_apply(c1["lat"], c1["U"], c1["psi"], RHO, 0.01, s_or)
    err = gu.rel_err(got, want)
    print("overlap apply prec %d rel err %.3e" % (prec, err))
    bound = {ovl.OVL_F32: 1e-5, ovl.OVL_F16: 3e-2, ovl.OVL_BF16: 2e-1}[prec]
    assert err < bound


def test_overlap_aliasing_rejected(c1):
    g = ovl.Geometry(c1["dims"])
    gauge = gu.make_gauge(g, c1["U"])
    s_lib = ovl.Sign(c1["lo"], c1["hi"], n=10)
    buf = gu.pack(g, c1["psi"], ovl.OVL_F64)
    with pytest.raises(ovl.OvlError) as e:
        ovl.ovl_overlap_apply(buf, buf, gauge, RHO, 0.01, s_lib, None, 0, ovl.OVL_F64, 1, None)
    assert e.value.name == "OVL_E_ALIAS"


@pytest.mark.parametrize("prec", [ovl.OVL_F64, ovl.OVL_F32, ovl.OVL_F16, ovl.OVL_BF16])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 4), (6, 6, 2, 10)])
def test_projection_tile_edges(prec, dims):
    """The matrix-core projection around its tiles: parities smaller than, equal
    to and not a multiple of the 32- and 64-site units (2^4: 8 half-sites, 4^4:
    128, 360), mode counts around 16-mode tiles, their groups of 1, 2, 4, 7 and
    8 waves and two groups of modes, one and two column tiles (8 and 9 vectors),
    eigenvalues of one sign and of both."""
    g = ovl.Geometry(dims)
    V = si.orthonormal_spinors(dims, 150, 17)
    vdev = _lowmodes_dev(g, V)
    Vm = V.reshape(150, -1)
    psi = np.stack([si.gaussian_spinor(dims, 800 + r) for r in range(12)])
    u = gu.UNIT_ROUNDOFF[prec]
    rng = np.random.default_rng(3)
    for ell, nrhs, signs in ((1, 1, 0), (3, 8, 1), (16, 9, -1), (17, 12, 0), (33, 2, 0), (49, 12, 1), (70, 5, 0),
                             (113, 12, 0), (128, 1, -1), (150, 12, 0)):
        lam = rng.uniform(0.1, 0.5, ell) * (signs if signs else rng.choice([-1.0, 1.0], ell))
        lm = ovl.LowModes(g, vdev, lam)
        inp = gu.pack(g, psi[:nrhs], prec, nrhs)
        h, w = gu.empty_field(g, prec, nrhs), gu.empty_field(g, prec, nrhs)
        ovl.ovl_lowmodes_project(lm, inp, h, w, prec, nrhs, None)
        x = np.reshape(gu.unpack(g, inp, prec, nrhs), (nrhs, -1))
        c = Vm[:ell].conj() @ x.T
        want_h = x - (Vm[:ell].T @ c).T
        want_w = (Vm[:ell].T @ (np.sign(lam)[:, None] * c)).T
        # FP64 sums of up to 150 terms of order one, then the storage rounding
        tol = 1e-13 if prec == ovl.OVL_F64 else 2 * u
        for dev, want in ((h, want_h), (w, want_w)):
            got = np.reshape(gu.unpack(g, dev, prec, nrhs), (nrhs, -1))
            assert np.max(np.abs(got - want)) <= tol * max(1.0, np.max(np.abs(want))), (ell, nrhs, signs)


@pytest.mark.parametrize("prec", [ovl.OVL_F64, ovl.OVL_F32, ovl.OVL_F16, ovl.OVL_BF16])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 6, 6, 10)])
def test_projection_of_few_vectors(prec, dims):
    """One and two vectors (no matrix instructions in the second reading) and
    the first batch past them: mode counts around the groups of 2, 4 and 8 that
    are read ahead, one sign or both, a site range with a remainder."""
    g = ovl.Geometry(dims)
    V = si.orthonormal_spinors(dims, 37, 19)
    vdev = _lowmodes_dev(g, V)
    Vm = V.reshape(37, -1)
    psi = np.stack([si.gaussian_spinor(dims, 900 + r) for r in range(3)])
    u = gu.UNIT_ROUNDOFF[prec]
    for ell in (1, 2, 3, 8, 9, 16, 17, 37):
        for nrhs in (1, 2, 3):
            for npos in {0, 1, ell // 2, ell}:
                lam = np.where(np.arange(ell) < npos, 0.2, -0.3)[::-1].copy()
                lm = ovl.LowModes(g, vdev, lam)
                inp = gu.pack(g, psi[:nrhs], prec, nrhs)
                h, w = gu.empty_field(g, prec, nrhs), gu.empty_field(g, prec, nrhs)
                ovl.ovl_lowmodes_project(lm, inp, h, w, prec, nrhs, None)
                x = np.reshape(gu.unpack(g, inp, prec, nrhs), (nrhs, -1))
                c = Vm[:ell].conj() @ x.T
                want_h = x - (Vm[:ell].T @ c).T
                want_w = (Vm[:ell].T @ (np.sign(lam)[:, None] * c)).T
                tol = 1e-13 if prec == ovl.OVL_F64 else 2 * u  # FP64 sums, then the storage rounding
                for dev, want in ((h, want_h), (w, want_w)):
                    got = np.reshape(gu.unpack(g, dev, prec, nrhs), (nrhs, -1))
                    assert np.max(np.abs(got - want)) <= tol * max(1.0, np.max(np.abs(want))), (ell, nrhs, npos)


@pytest.mark.parametrize("prec", [ovl.OVL_F64, ovl.OVL_F32, ovl.OVL_F16, ovl.OVL_BF16])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 4), (6, 6, 2, 10)])
def test_projection_waves_and_mode_groups(prec, dims):
    """The inner products where their split changes: 3, 5 and 6 waves and two
    groups of 5 of the matrix-core form; one and two vectors with 1 to 8 modes a
    wave, waves and groups that are not full, one to three groups of 64 modes."""
    g = ovl.Geometry(dims)
    V = si.orthonormal_spinors(dims, 150, 23)
    vdev = _lowmodes_dev(g, V)
    Vm = V.reshape(150, -1)
    psi = np.stack([si.gaussian_spinor(dims, 830 + r) for r in range(12)])
    u = gu.UNIT_ROUNDOFF[prec]
    rng = np.random.default_rng(4)
    for ell, nrhs in ((33, 4), (48, 12), (65, 3), (80, 12), (81, 5), (96, 9), (129, 12), (145, 8), (5, 1), (9, 2),
                      (20, 1), (33, 1), (57, 2), (64, 1), (64, 2), (65, 1), (66, 2), (128, 2), (129, 1), (143, 2)):
        lam = rng.uniform(0.1, 0.5, ell) * rng.choice([-1.0, 1.0], ell)
        lm = ovl.LowModes(g, vdev, lam)
        inp = gu.pack(g, psi[:nrhs], prec, nrhs)
        h, w = gu.empty_field(g, prec, nrhs), gu.empty_field(g, prec, nrhs)
        ovl.ovl_lowmodes_project(lm, inp, h, w, prec, nrhs, None)
        x = np.reshape(gu.unpack(g, inp, prec, nrhs), (nrhs, -1))
        c = Vm[:ell].conj() @ x.T
        want_h = x - (Vm[:ell].T @ c).T
        want_w = (Vm[:ell].T @ (np.sign(lam)[:, None] * c)).T
        tol = 1e-13 if prec == ovl.OVL_F64 else 2 * u  # FP64 sums, then the storage rounding
        for dev, want in ((h, want_h), (w, want_w)):
            got = np.reshape(gu.unpack(g, dev, prec, nrhs), (nrhs, -1))
            assert np.max(np.abs(got - want)) <= tol * max(1.0, np.max(np.abs(want))), (ell, nrhs)


@pytest.mark.parametrize("prec", [ovl.OVL_F64, ovl.OVL_F32, ovl.OVL_F16, ovl.OVL_BF16])
@pytest.mark.parametrize("dims", [(16, 16, 16, 8), (14, 16, 18, 10), (10, 16, 18, 10)])
def test_projection_of_few_vectors_on_larger_lattices(prec, dims):
    """One and two vectors where one load per thread is in flight (from 16384
    half-sites on: exactly, and with a remainder) and just below (14400), with one
    sign or both."""
    g = ovl.Geometry(dims)
    V = si.orthonormal_spinors(dims, 9, 29)
    vdev = _lowmodes_dev(g, V)
    Vm = V.reshape(9, -1)
    psi = np.stack([si.gaussian_spinor(dims, 860 + r) for r in range(2)])
    u = gu.UNIT_ROUNDOFF[prec]
    for ell, nrhs, npos in ((9, 1, 4), (9, 2, 1), (5, 2, 5), (1, 1, 0)):
        lam = np.where(np.arange(ell) < npos, 0.2, -0.3)[::-1].copy()
        lm = ovl.LowModes(g, vdev, lam)
        inp = gu.pack(g, psi[:nrhs], prec, nrhs)
        h, w = gu.empty_field(g, prec, nrhs), gu.empty_field(g, prec, nrhs)
        ovl.ovl_lowmodes_project(lm, inp, h, w, prec, nrhs, None)
        x = np.reshape(gu.unpack(g, inp, prec, nrhs), (nrhs, -1))
        c = Vm[:ell].conj() @ x.T
        want_h = x - (Vm[:ell].T @ c).T
        want_w = (Vm[:ell].T @ (np.sign(lam)[:, None] * c)).T
        tol = 1e-13 if prec == ovl.OVL_F64 else 2 * u  # FP64 sums, then the storage rounding
        for dev, want in ((h, want_h), (w, want_w)):
            got = np.reshape(gu.unpack(g, dev, prec, nrhs), (nrhs, -1))
            assert np.max(np.abs(got - want)) <= tol * max(1.0, np.max(np.abs(want))), (ell, nrhs, npos)
