"""GPU parity of the PTC layers and gradients against the FP64 oracle, and
the learned-preconditioner workflow (harvest, train, FGCR with fallback)."""
import ctypes

import numpy as np
import pytest

import synth_inputs as si
from oracle import dirac, ptc
from oracle.lattice import Lattice

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1106_4964_amd import ovl  # noqa: E402

import gpu_util as gu  # noqa: E402

DIMS = (6, 4, 4, 8)
F32 = ovl.OVL_F32


@pytest.fixture(scope="module")
def setup():
    lat = Lattice(DIMS)
    U = si.gauge_field(DIMS, 0.3, 31)
    g = ovl.Geometry(DIMS)
    gauge = gu.make_gauge(g, U, [(F32, 0)])
    return lat, U, g, gauge


def _w(seed, cout, cin, scale=0.3):
    rng = np.random.default_rng(seed)
    return scale * (rng.standard_normal((9, cout, cin, 4, 4)) + 1j * rng.standard_normal((9, cout, cin, 4, 4)))


def test_layer_with_wilson_weights_is_dslash(setup):
    lat, U, g, gauge = setup
    psi = si.gaussian_spinor(DIMS, 3)
    W = ptc.wilson_weights(0.1)
    out = gu.empty_field(g, F32)
    ovl.ovl_ptc_layer_forward(gauge, gu.pack(g, psi, F32), 1, out, 1, np.ascontiguousarray(W), None)
    got = gu.unpack(g, out, F32)
    assert gu.rel_err(got, dirac.wilson_dslash(lat, U, psi, 0.1)) < 2e-6


@pytest.mark.parametrize("cin,cout", [(1, 4), (4, 1), (2, 2)])
def test_layer_forward_and_backward(setup, cin, cout):
    lat, U, g, gauge = setup
    W = _w(cin * 10 + cout, cout, cin)
    phi = np.stack([si.gaussian_spinor(DIMS, 40 + i) for i in range(cin)])
    gout = np.stack([si.gaussian_spinor(DIMS, 50 + i) for i in range(cout)])
    Wc = np.ascontiguousarray(W)
    out = gu.empty_field(g, F32, cout)
    din = gu.pack(g, phi, F32, cin)
    ovl.ovl_ptc_layer_forward(gauge, din, cin, out, cout, Wc, None)
    got = gu.unpack(g, out, F32, cout).reshape(cout, g.N, 4, 3)
    want = ptc.forward(lat, U, W, phi)
    assert gu.rel_err(got, want) < 2e-6
    gin = gu.empty_field(g, F32, cin)
    gW = np.zeros_like(Wc)
    ovl.ovl_ptc_layer_backward(gauge, din, cin, gu.pack(g, gout, F32, cout), cout, Wc, gin, gW.ctypes.data, None)
    want_in, want_W = ptc.backward(lat, U, W, phi, gout)
    got_in = gu.unpack(g, gin, F32, cin).reshape(cin, g.N, 4, 3)
    assert gu.rel_err(got_in, want_in) < 2e-6
    # FP32 site sums against the FP64 oracle gradient
    assert gu.rel_err(gW, want_W) < 1e-4


@pytest.mark.parametrize("c12", [0, 1])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 6, 6, 10)])
def test_layer_channel_counts(dims, c12):
    """Every channel count the kernels are built for (all of 1..4 x 1..4 forward,
    products up to 4 backward), with fewer sites than a wave (2^4) and a last
    block that is not full, several blocks of the weight gradient and an odd
    number of values per lane in its wave sum (3 channels), on 18- and 12-real
    links."""
    lat = Lattice(dims)
    U = si.gauge_field(dims, 0.3, 12)
    g = ovl.Geometry(dims)
    gauge = gu.make_gauge(g, U, [(F32, c12)])
    phi = np.stack([si.gaussian_spinor(dims, 140 + i) for i in range(4)])
    gout = np.stack([si.gaussian_spinor(dims, 150 + i) for i in range(4)])
    for cin in range(1, 5):
        for cout in range(1, 5):
            W = np.ascontiguousarray(_w(cin * 10 + cout, cout, cin))
            out = gu.empty_field(g, F32, cout)
            din = gu.pack(g, phi[:cin], F32, cin)
            ovl.ovl_ptc_layer_forward(gauge, din, cin, out, cout, W, None)
            got = gu.unpack(g, out, F32, cout).reshape(cout, g.N, 4, 3)
            assert gu.rel_err(got, ptc.forward(lat, U, W, phi[:cin])) < 2e-6, (cin, cout)
            if cin * cout > 4:
                continue
            gin, gW = gu.empty_field(g, F32, cin), np.zeros_like(W)
            ovl.ovl_ptc_layer_backward(gauge, din, cin, gu.pack(g, gout[:cout], F32, cout), cout, W, gin, gW, None)
            want_in, want_W = ptc.backward(lat, U, W, phi[:cin], gout[:cout])
            assert gu.rel_err(gu.unpack(g, gin, F32, cin).reshape(cin, g.N, 4, 3), want_in) < 2e-6, (cin, cout)
            assert gu.rel_err(gW, want_W) < 1e-4, (cin, cout)


def _harvest(g, gauge, U, dims, cap):
    from oracle import dense  # noqa: F401
    s = ovl.Sign(0.4, 6.6, n=60)
    b = si.point_sources(dims)[:2]
    bd = gu.pack(g, b, ovl.OVL_F64, 2)
    x = gu.pack(g, np.zeros_like(b), ovl.OVL_F64, 2)
    hx = gu.empty_field(g, F32, cap)
    hb = gu.empty_field(g, F32, cap)
    opts = ovl.SolveOpts(ovl.OVL_F64, 0.0, 0, 1, 50, hx.data_ptr(), hb.data_ptr(), cap)
    st = ovl.SolveStats()
    ovl.ovl_cg_solve(x, bd, 2, gauge, 1.5, 0.05, s, None, 1e-10, 5000, opts, ctypes.byref(st), None)
    return s, hx, hb, st


def test_harvested_pairs_are_exact(setup):
    lat, U, g, gauge = setup
    s, hx, hb, st = _harvest(g, gauge, U, DIMS, 16)
    assert st.harvested == 16
    from oracle import sign
    so = sign.SignApprox(lam_max=6.6, eps=s.eps, coeffs=s.coeffs())
    X = gu.unpack(g, hx, F32, 16).reshape(16, g.N, 4, 3)
    B = gu.unpack(g, hb, F32, 16).reshape(16, g.N, 4, 3)
    for i in (0, 7, 15):
        assert gu.rel_err(B[i], sign.overlap_apply(lat, U, X[i], 1.5, 0.05, so)) < 1e-6


def test_harvest_stride_takes_every_kth_iteration(setup):
    """With harvest_stride k the pairs are those of inner iterations 0, k,
    2k, ...: bit-identical to the matching pairs of an every-iteration
    harvest of the same (deterministic) solve, and still exact pairs."""
    lat, U, g, gauge = setup
    s = ovl.Sign(0.4, 6.6, n=60)
    b = si.point_sources(DIMS)[:2]
    out = {}
    for stride, cap in ((1, 12), (5, 4)):
        x = gu.pack(g, np.zeros_like(b), ovl.OVL_F64, 2)
        hx, hb = gu.empty_field(g, F32, cap), gu.empty_field(g, F32, cap)
        opts = ovl.SolveOpts(ovl.OVL_F64, 0.0, 0, 1, 50, hx.data_ptr(), hb.data_ptr(), cap)
        opts.harvest_stride = stride
        st = ovl.SolveStats()
        ovl.ovl_cg_solve(x, gu.pack(g, b, ovl.OVL_F64, 2), 2, gauge, 1.5, 0.05, s, None, 1e-10, 5000, opts,
                         ctypes.byref(st), None)
        assert st.harvested == cap
        out[stride] = (gu.unpack(g, hx, F32, cap), gu.unpack(g, hb, F32, cap))
    # two rhs per iteration: pair 2 i + r of stride 5 is iteration 5 i, pair 2 (5 i) + r of stride 1
    for k5, k1 in ((0, 0), (1, 1), (2, 10), (3, 11)):
        assert np.array_equal(out[5][0][k5], out[1][0][k1]) and np.array_equal(out[5][1][k5], out[1][1][k1])
    from oracle import sign
    so = sign.SignApprox(lam_max=6.6, eps=s.eps, coeffs=s.coeffs())
    assert gu.rel_err(out[5][1][3], sign.overlap_apply(lat, U, out[5][0][3], 1.5, 0.05, so)) < 1e-6


def test_fgcr_batch_matches_single_rhs(setup):
    """The lockstep batched FGCR (3 rhs, with a network and with M = 1)
    gives each rhs the solution of its own single-rhs FGCR solve, both at the
    FP64 true residual 1e-10."""
    lat, U, g, gauge = setup
    s = ovl.Sign(0.4, 6.6, n=60)
    net = ovl.Net(g, 4)
    w1, w2 = _w(41, 4, 1, 0.005), _w(42, 1, 4, 0.005)  # M: 1/rho plus a small learned-like part
    w1[0, 0, 0] += np.eye(4)
    w2[0, 0, 0] += np.eye(4) / 1.5
    net.set_weights(w1, w2)
    b = si.point_sources(DIMS)[[3, 9, 5]]
    for M in (net, None):
        opts = ovl.SolveOpts(F32, 1e-5, 0, 1, 50, None, None, 0)
        x = gu.pack(g, np.zeros_like(b), ovl.OVL_F64, 3)
        st = ovl.SolveStats()
        rc = ovl.ovl_fgcr_solve(x, gu.pack(g, b, ovl.OVL_F64, 3), 3, gauge, 1.5, 0.05, s, None, M, 8, 1e-10, 3000,
                                opts, ctypes.byref(st), None)
        print("batched FGCR (%s): %d iterations, fallback %d" % ("net" if M else "M=1", st.iterations,
                                                                 st.fallback_used))
        assert rc == 0 and st.fallback_used == 0 and max(st.true_residual[:3]) <= 1e-10
        xb = gu.unpack(g, x, ovl.OVL_F64, 3)
        for r in range(3):
            x1 = gu.pack(g, np.zeros_like(b[r]), ovl.OVL_F64, 1)
            s1 = ovl.SolveStats()
            assert ovl.ovl_fgcr_solve(x1, gu.pack(g, b[r], ovl.OVL_F64, 1), 1, gauge, 1.5, 0.05, s, None, M, 8, 1e-10,
                                      3000, opts, ctypes.byref(s1), None) == 0
            assert gu.rel_err(xb[r], gu.unpack(g, x1, ovl.OVL_F64, 1)) < 1e-7


def test_training_reduces_loss_and_fgcr(setup):
    lat, U, g, gauge = setup
    npairs = 48
    s, hx, hb, st = _harvest(g, gauge, U, DIMS, npairs)
    assert st.harvested == npairs
    net = ovl.Net(g, 4)
    rng = np.random.default_rng(5)
    w1 = 0.05 * (rng.standard_normal((9, 4, 1, 4, 4)) + 1j * rng.standard_normal((9, 4, 1, 4, 4)))
    w2 = 0.05 * (rng.standard_normal((9, 1, 4, 4, 4)) + 1j * rng.standard_normal((9, 1, 4, 4, 4)))
    w1[0, 0, 0] += np.eye(4)
    w2[0, 0, 0] += np.eye(4) / 1.5
    net.set_weights(w1, w2)
    epochs = 6
    order = np.concatenate([rng.permutation(npairs) for _ in range(epochs)]).astype(np.int32)
    hist = np.zeros(epochs)
    ovl.ovl_net_train(net, gauge, hb, hx, npairs, epochs, 8, 2e-3, order, hist, None)
    print("training loss per epoch", hist)
    assert np.all(np.isfinite(hist)) and hist[-1] < hist[0]
    # FGCR with the trained net, with M = 1, and with a broken net (fallback)
    b = si.point_sources(DIMS)[[3, 9]]
    res = {}
    for name, M in [("net", net), ("identity", None)]:
        x = gu.pack(g, np.zeros_like(b), ovl.OVL_F64, 2)
        fst = ovl.SolveStats()
        rc = ovl.ovl_fgcr_solve(x, gu.pack(g, b, ovl.OVL_F64, 2), 2, gauge, 1.5, 0.05, s, None, M, 16, 1e-10, 3000,
                                ovl.SolveOpts(F32, 1e-5, 0, 1, 50, None, None, 0), ctypes.byref(fst), None)
        assert rc == 0 and max(fst.true_residual[:2]) <= 1e-10
        res[name] = (fst.iterations, fst.fallback_used, fst.seconds)
    print("fgcr iterations (net, identity):", res)
    bad = ovl.Net(g, 4)
    bad.set_weights(np.full_like(w1, np.nan), w2)
    x = gu.pack(g, np.zeros_like(b), ovl.OVL_F64, 2)
    fst = ovl.SolveStats()
    rc = ovl.ovl_fgcr_solve(x, gu.pack(g, b, ovl.OVL_F64, 2), 2, gauge, 1.5, 0.05, s, None, bad, 16, 1e-10, 3000,
                            ovl.SolveOpts(F32, 1e-5, 0, 1, 50, None, None, 0), ctypes.byref(fst), None)
    assert rc == 0 and fst.fallback_used == 1 and max(fst.true_residual[:2]) <= 1e-10


def test_trained_net_gain_over_identity():
    """The trained network as right preconditioner of FGCR needs fewer D(m)
    applications than the same FGCR with M = 1 (8^4, m = 0.05, 12 point
    sources, low modes projected).  Training pairs: Gaussian x with
    b = D(m) x in FP32.  Both solves reach the FP64 true residual 1e-10
    without falling back to CG."""
    dims = (8, 8, 8, 8)
    rho, mass = 1.5, 0.05
    U = si.gauge_field(dims, 0.25, 3)
    g = ovl.Geometry(dims)
    gauge = gu.make_gauge(g, U, [(F32, 0)])
    v0 = gu.pack(g, si.gaussian_spinor(dims, 7), ovl.OVL_F64)
    lam = ctypes.c_double()
    ovl.ovl_hw_bound(gauge, rho, v0, 60, ctypes.byref(lam), None, None, None)
    lam_max = lam.value * (1 + 1e-6)
    ell, m_ = 8, 24
    V = gu.pack(g, np.stack([si.gaussian_spinor(dims, 900 + i) for i in range(m_)]), ovl.OVL_F64, m_)
    lams = np.zeros(ell)
    est = ovl.EigStats()
    assert ovl.ovl_hw_eigs(gauge, rho, ell, m_, V, lams, lam_max, 1e-10, 40, 30, ctypes.byref(est), None) == 0
    lm = ovl.LowModes(g, V, lams)
    sgn = ovl.Sign(abs(lams[-1]), lam_max, delta=1e-8)
    npairs = 192
    X = gu.pack(g, np.stack([si.gaussian_spinor(dims, 5000 + i) for i in range(npairs)]), F32, npairs)
    B = torch.empty_like(X)
    vb = g.spinor_bytes(F32)
    for i0 in range(0, npairs, 12):
        ovl.ovl_overlap_apply(B[i0 * vb:], X[i0 * vb:], gauge, rho, mass, sgn, lm, 0, F32, 12, None)
    net = ovl.Net(g, 4)
    rng = np.random.default_rng(5)
    w1 = 0.02 * (rng.standard_normal((9, 4, 1, 4, 4)) + 1j * rng.standard_normal((9, 4, 1, 4, 4)))
    w2 = 0.02 * (rng.standard_normal((9, 1, 4, 4, 4)) + 1j * rng.standard_normal((9, 1, 4, 4, 4)))
    w1[0, 0, 0] += np.eye(4)
    w2[0, 0, 0] += np.eye(4) / rho
    net.set_weights(w1, w2)
    epochs = 20
    order = np.concatenate([rng.permutation(npairs) for _ in range(epochs)]).astype(np.int32)
    hist = np.zeros(epochs)
    ovl.ovl_net_train(net, gauge, B, X, npairs, epochs, 8, 1e-3, order, hist, None)
    assert hist[-1] < 0.25 * hist[0]
    b = si.point_sources(dims)
    res = {}
    for name, M in [("net", net), ("identity", None)]:
        x = gu.pack(g, np.zeros_like(b), ovl.OVL_F64, 12)
        st = ovl.SolveStats()
        rc = ovl.ovl_fgcr_solve(x, gu.pack(g, b, ovl.OVL_F64, 12), 12, gauge, rho, mass, sgn, lm, M, 32, 1e-10, 20000,
                                ovl.SolveOpts(F32, 1e-4, 0, 1, 60, None, None, 0), ctypes.byref(st), None)
        assert rc == 0 and st.fallback_used == 0 and max(st.true_residual[:12]) <= 1e-10
        res[name] = (st.iterations, st.sign_applies)
    print("FGCR(32) iterations / sign applies, trained net vs M = 1:", res, "loss", hist[0], "->", hist[-1])
    assert res["net"][1] < 0.8 * res["identity"][1]
