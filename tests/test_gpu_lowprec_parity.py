"""Element-wise parity of the low-precision batched overlap operator.

The operator the benchmark times is D(m) and D(m)^dag (eq. 3, 8) on 12
right-hand sides with F16 storage (FP32 arithmetic), low modes projected
exactly (eq. 6-7) and the polynomial sign evaluated by the Clenshaw
recursion (eq. 4-5).  Here every one of the 12 outputs is compared with the
FP64 oracle on the same coefficients and low modes, site by site: the error
of a vector is max |got - want| / max |want|.  BF16 storage is checked the
same way.  The bounds are a stated multiple of the errors measured on
MI355X (recorded next to each bound).

Low modes: at 4^4 the 20 eigenvectors of H_w closest to zero from the
oracle's dense eigendecomposition (real low modes of the interacting
field); at 8^4 24 orthonormal vectors with made-up eigenvalues, so the
projection kernels see many tiles (the operator is the same formula for any
orthonormal basis).  The oracle never takes an input from the GPU path.
"""
import ctypes

import numpy as np
import pytest

import synth_inputs as si
from oracle import dense, sign, solvers, dirac
from oracle.lattice import Lattice

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1106_4964_amd import ovl  # noqa: E402

import gpu_util as gu  # noqa: E402

RHO, MASS, R = 1.5, 0.01, 12
F16, BF16, F64 = ovl.OVL_F16, ovl.OVL_BF16, ovl.OVL_F64

# Element-wise bounds, max over the 12 vectors of max|got - want| / max|want|,
# set at about 2.5x the largest error measured on MI355X over the 12 vectors
# and both D(m) and D(m)^dag:
#   4^4, n = 120, l = 20:  F16 9.3e-4, BF16 7.8e-3
#   8^4, n = 100, l = 24:  F16 1.0e-3, BF16 8.7e-3
BOUND_4444 = {F16: 2.5e-3, BF16: 2e-2}
BOUND_8888 = {F16: 2.5e-3, BF16: 2e-2}


def _elementwise(got, want):
    return [gu.max_rel_err(got[r], want[r]) for r in range(len(want))]


@pytest.fixture(scope="module")
def c1():
    dims = (4, 4, 4, 4)
    lat = Lattice(dims)
    U = si.gauge_field(dims, 0.3, 1)
    H = dense.dense_hw(lat, U, RHO)
    V, lam = dense.lowmodes(lat, H, 20)
    hi = dense.spectrum_bounds(H)[1] * 1.0001
    so = sign.make_sign(abs(lam[-1]), hi, 120)
    psi = np.stack([si.gaussian_spinor(dims, 900 + r) for r in range(R)])
    want = {d: np.stack([sign.overlap_apply(lat, U, psi[r], RHO, MASS, so, V, lam, dagger=bool(d)) for r in range(R)])
            for d in (0, 1)}
    return dict(dims=dims, U=U, V=V, lam=lam, lo=abs(lam[-1]), hi=hi, psi=psi, want=want)


@pytest.mark.parametrize("dagger", [0, 1])
@pytest.mark.parametrize("prec", [F16, BF16])
def test_overlap_12rhs_real_lowmodes_4444(c1, prec, dagger):
    g = ovl.Geometry(c1["dims"])
    gauge = gu.make_gauge(g, c1["U"], [(prec, 1)])
    lm = ovl.LowModes(g, gu.pack(g, c1["V"], F64, len(c1["V"])), c1["lam"])
    s = ovl.Sign(c1["lo"], c1["hi"], n=120)
    x = gu.pack(g, c1["psi"], prec, R)
    y = gu.empty_field(g, prec, R)
    ovl.ovl_overlap_apply(y, x, gauge, RHO, MASS, s, lm, dagger, prec, R, None)
    errs = _elementwise(gu.unpack(g, y, prec, R), c1["want"][dagger])
    print("4^4 D(m)%s prec %d, 12 rhs, l = 20, n = 120: element-wise errors %s"
          % ("^dag" if dagger else "", prec, " ".join("%.2e" % e for e in errs)))
    assert max(errs) < BOUND_4444[prec]


@pytest.fixture(scope="module")
def c8():
    """8^4, c = 0.25: the 12 inputs are psi_a + c_r psi_b (c_r = r - 5.5), so
    the oracle's two outputs give all twelve expected vectors by linearity."""
    dims = (8, 8, 8, 8)
    lat = Lattice(dims)
    U = si.gauge_field(dims, 0.25, 4)
    ell = 24
    V = si.orthonormal_spinors(dims, ell, seed=31)
    lam = np.concatenate([np.linspace(0.3, 0.45, ell // 2), -np.linspace(0.31, 0.46, ell // 2)])
    hi, _, _ = solvers.lanczos_bound(lambda v: dirac.hw_apply(lat, U, v, RHO), si.gaussian_spinor(dims, 17), 60)
    hi *= 1.001
    lo = 0.35  # below the smallest |lambda| of these near-unit fields
    so = sign.make_sign(lo, hi, 100)
    pa, pb = si.gaussian_spinor(dims, 950), si.gaussian_spinor(dims, 951)
    coef = np.arange(R) - 5.5
    psi = pa[None] + coef[:, None, None, None] * pb[None]
    want = {}
    for d in (0, 1):
        oa = sign.overlap_apply(lat, U, pa, RHO, MASS, so, V, lam, dagger=bool(d))
        ob = sign.overlap_apply(lat, U, pb, RHO, MASS, so, V, lam, dagger=bool(d))
        want[d] = oa[None] + coef[:, None, None, None] * ob[None]
    return dict(dims=dims, U=U, V=V, lam=lam, lo=lo, hi=hi, psi=psi, want=want)


@pytest.mark.parametrize("dagger", [0, 1])
@pytest.mark.parametrize("prec", [F16, BF16])
def test_overlap_12rhs_projected_8888(c8, prec, dagger):
    g = ovl.Geometry(c8["dims"])
    gauge = gu.make_gauge(g, c8["U"], [(prec, 1)])
    lm = ovl.LowModes(g, gu.pack(g, c8["V"], F64, len(c8["V"])), c8["lam"])
    s = ovl.Sign(c8["lo"], c8["hi"], n=100)
    x = gu.pack(g, c8["psi"], prec, R)
    y = gu.empty_field(g, prec, R)
    ovl.ovl_overlap_apply(y, x, gauge, RHO, MASS, s, lm, dagger, prec, R, None)
    errs = _elementwise(gu.unpack(g, y, prec, R), c8["want"][dagger])
    print("8^4 D(m)%s prec %d, 12 rhs, l = 24, n = 100: element-wise errors %s"
          % ("^dag" if dagger else "", prec, " ".join("%.2e" % e for e in errs)))
    assert max(errs) < BOUND_8888[prec]


def _f16(a):
    """The nearest F16 numbers, as complex128 and as the float64 reals."""
    h = np.ascontiguousarray(a).view(np.float64).astype(np.float16).astype(np.float64)
    return h.view(np.complex128), h


def _hw_hops_in_turn(lat, U, psi, rho):
    """H_w of F16 numbers in FP32 FMAs, each hop added to the sum as it is formed
    (forward, backward, direction by direction), then rounded to F16.  Arrays are
    float32 (re, im) pairs; the float64 product of two float32 is exact."""
    f4 = np.float32

    def fma(x, y, z):
        return (x.astype(np.float64) * y + z).astype(f4)

    def parts(v):
        return np.stack([v.real, v.imag], -1).astype(f4)

    p, u = parts(psi.reshape(lat.shape + (4, 3))), parts(U.reshape(lat.shape + (4, 3, 3)))
    acc = np.zeros_like(p)
    half = f4(-0.5)
    turn = {1: lambda v: v, -1: lambda v: -v, 1j: lambda v: np.stack([-v[..., 1], v[..., 0]], -1),
            -1j: lambda v: np.stack([v[..., 1], -v[..., 0]], -1)}
    for mu in range(4):
        gam = dirac.GAMMA[mu]
        for s in (-1, 1):  # forward (1 - gamma), backward (1 + gamma)
            n = np.roll(p, s, axis=3 - mu)
            link = u[..., mu, :, :, :] if s < 0 else np.roll(u[..., mu, :, :, :], 1, axis=3 - mu)
            w = []
            for k in range(2):
                j = int(np.argmax(np.abs(gam[k])))
                h = n[..., k, :, :] + turn[complex(s * gam[k, j])](n[..., j, :, :])
                rows = []
                for a in range(3):
                    re = im = np.zeros(lat.shape, f4)
                    for b in range(3):
                        v = link[..., a, b, :] if s < 0 else link[..., b, a, :] * np.array([1, -1], f4)
                        re, im = fma(v[..., 0], h[..., b, 0], re), fma(v[..., 0], h[..., b, 1], im)
                        re, im = fma(-v[..., 1], h[..., b, 1], re), fma(v[..., 1], h[..., b, 0], im)
                    rows.append(np.stack([re, im], -1))
                w.append(np.stack(rows, -2))
            for k in range(4):
                if k < 2:
                    add = w[k]
                else:  # gamma chi = s chi for chi = (1 + s gamma) psi
                    j = int(np.argmax(np.abs(gam[k, :2])))
                    add = turn[complex(s * gam[k, j])](w[j])
                acc[..., k, :, :] = fma(add, half, acc[..., k, :, :])
    acc = fma(p, f4(4.0 - rho), acc)
    acc[..., 2:, :, :] *= f4(-1)
    return acc.astype(np.float16).astype(np.float64).reshape(-1)


def test_f16_stencil_rounds_no_more_than_hops_added_in_turn():
    """H_w at F16 storage with every input an F16 number: the stored reals that
    are not the rounding of the exact value (the FP64 stencil on the same
    numbers) count the FP32 arithmetic's roundings, which the storage rounding
    hides from the usual error.  No more than the plainest FP32 form leaves on
    the same numbers, within three standard deviations of its count."""
    dims = (8, 8, 12, 16)
    lat = Lattice(dims)
    g = ovl.Geometry(dims)
    wrong = plain = 0
    for seed in range(6):
        U = _f16(si.gauge_field(dims, 0.25, 30 + seed))[0]
        gauge = gu.make_gauge(g, U, [(F16, 0)])
        psi = np.stack([_f16(si.gaussian_spinor(dims, 100 * seed + r))[0] for r in range(R)])
        got = {}
        for prec in (F16, F64):
            out = gu.empty_field(g, prec, R)
            ovl.ovl_hw_apply(out, gu.pack(g, psi, prec, R), gauge, RHO, prec, R, None)
            got[prec] = np.ascontiguousarray(gu.unpack(g, out, prec, R))
        want = _f16(got[F64])[1].reshape(R, -1)
        wrong += int(np.count_nonzero(got[F16].view(np.float64).reshape(R, -1) != want))
        for r in range(R):
            plain += int(np.count_nonzero(_hw_hops_in_turn(lat, U, psi[r], RHO) != want[r]))
    print("F16 H_w: reals off the exact value's rounding %d, hops in turn %d of %d" % (wrong, plain, 6 * R * 24 * g.N))
    assert wrong <= plain + 3 * np.sqrt(plain)
