"""The FP32 Norton roots, which start from a table per family and have no
history: the local law against the oracle for exponents over the table's
range and below it, for families that differ, for overstresses on both
sides of the crossover and far from it, and where the lanes of a wave are
not all in use."""
import dataclasses

import numpy as np
import pytest

import oracle
import rvegen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
cp = pytest.importorskip("paper_2402_09996_amd")

# name: (slip n, K), (twin n, K), eta, twin mode
LAWS = {
    "linear": ((1.0, 2000.0), (1.0, 2000.0), None, 0),
    "below the table": ((1.3, 900.0), (1.3, 900.0), None, 0),
    "least exponent": ((1.5, 600.0), (1.5, 600.0), None, 0),
    "n = 3": ((3.0, 120.0), (3.0, 120.0), None, 0),
    "n = 10": (None, None, None, 1),
    "n = 30": ((30.0, 14.0), (30.0, 14.0), None, 0),
    "two families": ((10.0, 25.0), (4.0, 60.0), None, 1),
    "Norton side": ((10.0, 80.0), (10.0, 80.0), None, 0),
    "viscous side": ((10.0, 4.0), (10.0, 4.0), 4.0e4, 0),
    "unregularized": ((2.0, 2000.0), (2.0, 2000.0), 0.0, 0),
}


def _relerr(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def _inputs(kind, shape, twins):
    C, law = rvegen.config_law()
    slip, twin, eta, law.twin_mode = LAWS[kind]
    if slip:
        law.slip = dataclasses.replace(law.slip, n=slip[0], K=slip[1])
        law.twin = dataclasses.replace(law.twin, n=twin[0], K=twin[1])
    if eta is not None:
        law.eta = eta
    if law.twin_mode:
        law.K_c, law.f_m = 1.45, 0.8
    w = rvegen.Workload("roots", rvegen.make_rve(shape, 4, 5), rvegen.config_systems(twins), C, law,
                        rvegen.uniaxial_path(1e-3, 1))
    rng = np.random.default_rng(3)
    nv, S = int(np.prod(shape)), w.systems.family.shape[0]
    e0 = rng.standard_normal((nv, 6)) * 1e-3
    ep = rng.standard_normal((nv, 6)) * 2e-4
    ep[:, :3] -= ep[:, :3].mean(axis=1, keepdims=True)
    v = rng.random((nv, S)) * 2e-3
    al = rng.standard_normal((nv, S)) * 1e-3
    return w, e0, e0 + rng.standard_normal((nv, 6)) * 4e-4, np.hstack([ep, v, al])


def _oracle(w, e0, e1, st0, dt, M):
    mat = oracle.Material(w.rve.euler, w.C, w.systems.n_miller, w.systems.l_miller, w.systems.family,
                          w.systems.tau0, w.law)
    y1, sig = mat.update(w.rve.labels.ravel(), oracle.to_mandel(e0), oracle.to_mandel(e1),
                         np.hstack([oracle.to_mandel(st0[:, :6]), st0[:, 6:]]), dt, M)
    return np.hstack([oracle.from_mandel(y1[:, :6]), y1[:, 6:]]), oracle.from_mandel(sig)


@pytest.mark.parametrize("kind", list(LAWS))
@pytest.mark.parametrize("shape,twins", [((4, 9, 9), True), ((2, 3, 3), False)])
def test_fp32_local_law_matches_oracle(kind, shape, twins):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("case", kind, shape, flush=True)
    w, e0, e1, st0 = _inputs(kind, shape, twins)
    S, nv = w.systems.family.shape[0], int(np.prod(shape))
    ref_st, ref_sig = _oracle(w, e0, e1, st0, 0.4, 8)
    assert (np.abs(ref_st[:, 6:6 + S] - st0[:, 6:6 + S]).max(axis=1) > 0).mean() > 0.5    # plastic

    def grid(a):
        return torch.from_numpy(np.ascontiguousarray(a.T.reshape((a.shape[1],) + shape)))

    s = cp.Solver(cp.Problem.from_workload(w), precision="fp32")
    st1, sg = s.constitutive(grid(e0), grid(e1), grid(st0), 0.4, 8)
    st1 = st1.cpu().numpy().reshape(6 + 2 * S, nv).T
    # the bounds of the other FP32 comparisons of the local law
    assert _relerr(sg.cpu().numpy().reshape(6, nv).T, ref_sig) < 2e-5
    for a, b in ((0, 6), (6, 6 + S), (6 + S, 6 + 2 * S)):
        assert _relerr(st1[:, a:b], ref_st[:, a:b]) < 2e-4


def _plain(n, K, eta, shape, strain, seed=7):
    """Local law without initial resistance and hardening from rest, to
    deviatoric strains of that size (FP32 values): the solver's and the
    oracle's state after it and the stress."""
    C, law = rvegen.config_law()
    law.slip = dataclasses.replace(law.slip, n=n, K=K, Q=0.0, c=0.0, d=0.0)
    law.eta = eta
    w = rvegen.Workload("plain", rvegen.make_rve(shape, 8, 5), rvegen.config_systems(False, 0.0, 0.0), C, law,
                        rvegen.uniaxial_path(1e-3, 1))
    rng = np.random.default_rng(seed)
    nv = int(np.prod(shape))
    e1 = rng.standard_normal((nv, 6))
    e1[:, :3] -= e1[:, :3].mean(axis=1, keepdims=True)
    e1 = (e1 * strain).astype(np.float32)
    st0 = np.zeros((nv, 30))
    ref_st, ref_sig = _oracle(w, 0.0 * e1, e1.astype(np.float64), st0, 1e-6, 1)

    def grid(a):
        return torch.from_numpy(np.ascontiguousarray(a.T.reshape((a.shape[1],) + shape)))

    s = cp.Solver(cp.Problem.from_workload(w), precision="fp32")
    st1, sg = s.constitutive(grid(0.0 * e1), grid(e1), grid(st0), 1e-6, 1)
    return (st1.cpu().numpy().reshape(30, nv).T.astype(np.float64), ref_st,
            sg.cpu().numpy().reshape(6, nv).T.astype(np.float64), ref_sig)


# Overstresses a tenth to a third above K, of which the rate is that share:
# rounding of the overstress, up to 2e-6 of it, is 2e-5 of the rate, and the
# root's 1.1e-7 adds 1e-6 whatever the exponent.
@pytest.mark.parametrize("n", [50.0, 100.0, 200.0, 400.0])
def test_fp32_roots_of_large_exponents_match_oracle(n):
    print("case", n, flush=True)
    K, eta = 60.0, 10.0
    st, ref, _, _ = _plain(n, K, eta, (8, 16, 16), 3e-4)
    v, vr = st[:, 6:18], ref[:, 6:18]
    g = np.maximum(vr, 0.0) * 6e6           # the last stage's: the others are below K
    share = (g ** (1.0 / n) * K + eta * g) / K
    sel = (share > 1.1) & (share < 1.35)
    assert sel.sum() > 500
    assert np.abs(v[sel] / vr[sel] - 1.0).max() < 3e-5


# Overstresses down to the least FP32 values: the bound of the other
# comparisons, beside rounding of o - K y (2e-7 of the stress, over eta) and
# of the slip (1e-42).
@pytest.mark.parametrize("n", [1.0, 10.0])
@pytest.mark.parametrize("strain", [1e-25, 1e-32, 1e-36, 1e-38, 1e-43])
def test_fp32_vanishing_overstress(n, strain):
    print("case", n, strain, flush=True)
    st, ref, sig, ref_sig = _plain(n, 2000.0, 1e4, (2, 4, 4), strain)
    assert np.isfinite(st).all() and np.isfinite(sig).all()
    assert np.abs(st[:, 6:18] - ref[:, 6:18]).max() <= (2e-4 * ref[:, 6:18].max() + 1e-42 +
                                                             2e-7 * np.abs(ref_sig).max() / 1e4 * 1e-6)
    assert np.abs(sig - ref_sig).max() <= 2e-5 * np.abs(ref_sig).max() + 1e-38


# n_newton counts the steps of the root solves: two for each with an exponent
# of 1, where they start from the smaller of o/K and o/eta and a second step
# finds nothing left; one, but for few, from the table.  Groups of 64 lanes
# that are full and partly empty.
@pytest.mark.parametrize("shape", [(2, 2, 4), (3, 3, 3), (4, 8, 8)])
def test_fp32_step_count(shape):
    for n, K, lo, hi in ((1.0, 2000.0, 2.0, 2.0), (10.0, 10.0, 1.0, 1.05)):
        print("case", shape, n, flush=True)
        C, law = rvegen.config_law()
        law.slip = dataclasses.replace(law.slip, n=n, K=K)
        path = rvegen.LoadPath(t=np.array([0.0, 0.4]), strain_ctrl=np.ones((1, 6), np.uint8),
                               target=4e-3 * np.array([[1.0, -0.45, -0.55, 0.12, -0.2, 0.31]]))
        w = rvegen.Workload("count", rvegen.make_rve(shape, 1, 5), rvegen.config_systems(False), C, law, path)
        R = cp.Solver(cp.Problem.from_workload(w), precision="fp32", tol=1e-4, rk4_M=4).run(w.path)
        assert R["n_active"][0] > 0
        ratio = R["n_newton"][0] / R["n_active"][0]
        assert lo <= ratio <= hi
