"""Coarse GMRES over more steps than it needs, and beyond a wave's width of them."""
import numpy as np
import pytest

from gpu_common import case, coarse_to_lex, dev, host, lex_to_coarse, need_gpu
from oracle import clover as oclover
from oracle import dirac, krylov, mg
from synth import random_links, random_spinors, random_test_vectors, seed_for

pytestmark = pytest.mark.gpu
DIMS, BLOCK = (8, 8, 8, 8), (4, 4, 4, 4)


_LEVEL = {}


def _mg(ntv):
    qmg = need_gpu()
    U = random_links(DIMS, 0.5, seed_for(2, "U"))
    W = random_test_vectors(DIMS, ntv, seed_for(2, "W"))
    if ntv not in _LEVEL:
        _LEVEL[ntv] = mg.TwoLevel(dirac.Operator(U, -0.8, oclover.clover_term(U, 1.0)), list(W), BLOCK)
    lat = qmg.Lattice(DIMS, BLOCK)
    lat.set_gauge(dev(U), -0.8, 1.0)
    lat.set_test_vectors(lat.pack(dev(W)), ntv)
    return qmg, lat, _LEVEL[ntv], lat.coarse_site_order()


# 65 and 80 steps: the last one's coefficients take more than one wave.  The shift lies inside
# the spectrum (singular values of the coarse operator from 5e-5 to 6.6), so the residual is
# still near 0.1 and well above rounding; GMRES minimises it, so an error of delta in the
# coefficients changes it by order delta^2 / residual and 1e-9 holds with a wide margin
@pytest.mark.parametrize("iters", [65, 80])
def test_device_gmres_many_steps(iters):
    case("device gmres %d steps" % iters)
    qmg, lat, h, _ = _mg(24)
    r = random_spinors(DIMS, 1, 41)
    prm = qmg.default_params(coarse_maxiter=iters, coarse_tol=0.0, nu_post=0)
    z = host(lat.unpack(lat.vcycle(lat.field(1), lat.pack(dev(r)), [3.0], 1, prm), 1))
    rc, y = mg.restrict(h.P, r[0], BLOCK), mg.restrict(h.P, z[0], BLOCK)
    _, _, best = krylov.gmres(lambda v: h.coarse.apply(v, 3.0), rc, iters)
    got = np.linalg.norm(rc - h.coarse.apply(y, 3.0))
    assert abs(got - best) < 1e-9 * np.linalg.norm(rc)


def _solve(lat, order, r, taus, iters, tol, prec):
    real = np.float64 if prec == "f64" else np.float32
    rd = dev(lex_to_coarse(r, order).view(np.float64).astype(real))
    out = lat.coarse_solve(lat.coarse(len(taus), prec), rd, taus, len(taus), iters, tol, prec)
    return coarse_to_lex(host(out).view(real).astype(np.float64).view(np.complex128), order, r.shape[-1] // 2)


def _rhs(order, ntv, nrhs, seed=8):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((nrhs, len(order), 2 * ntv)) + 1j * rng.standard_normal((nrhs, len(order), 2 * ntv))


# Backward error of a solve whose Krylov space is exhausted after 15 (first shift) and 60
# steps: ||r - A y|| <= tol (||A|| ||y|| + ||r||), ||A|| <= 6.1 here, with the relative error of
# one coarse apply as tol: 9 * 48 products at 2^-53 and 2^-24, and in BF16 blocks held to 2^-9
_APPLY_TOL = {"f64": 1e-13, "f32": 2.6e-5, "bf16": 2e-2}


def _backward(h, r, y, tau):
    return np.linalg.norm(r - h.coarse.apply(y, tau)) / (6.1 * np.linalg.norm(y) + np.linalg.norm(r))


# host-driven, three right-hand sides, one of them zero; as many steps as the default
# coarse_maxiter and several times that
@pytest.mark.parametrize("prec,iters", [("f32", 50), ("f32", 150), ("bf16", 60), ("f64", 120), ("f64", 200)])
def test_coarse_solve_past_convergence(prec, iters):
    case("coarse solve %s %d steps" % (prec, iters))
    _, lat, h, order = _mg(24)
    r = _rhs(order, 24, 3)
    r[1] = 0.0
    taus = [0.02, 0.1, 2.5]
    y = _solve(lat, order, r, taus, iters, 0.0, prec)
    assert not y[1].any()
    for k in (0, 2):
        assert _backward(h, r[k], y[k], taus[k]) < _APPLY_TOL[prec]


# one right-hand side reaches the tolerance in a few steps, the other never does: the first
# gets the solution it gets alone (the same steps; the batch changes the order of no sum
# beyond those of the coarse apply), the second the residual it gets alone
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 2.6e-5)])
def test_coarse_solve_mixed_batch(prec, tol):
    case("coarse solve mixed batch %s" % prec)
    _, lat, h, order = _mg(24)
    r, taus, iters = _rhs(order, 24, 2), [0.02, 3.0], 120
    both = _solve(lat, order, r, taus, iters, 1e-5, prec)
    alone = [_solve(lat, order, r[k:k + 1], taus[k:k + 1], iters, 1e-5, prec)[0] for k in range(2)]
    assert np.linalg.norm(both[0] - alone[0]) < tol * np.linalg.norm(alone[0])
    res = [np.linalg.norm(r[1] - h.coarse.apply(y, 3.0)) / np.linalg.norm(r[1]) for y in (both[1], alone[1])]
    assert res[1] < 0.2 and abs(res[0] - res[1]) < 1e-3 * res[1]


# the same on the device (V-cycle without smoothing, fixed steps): P^H of its result is y
@pytest.mark.parametrize("prec,iters", [("f32", 50), ("f32", 100), ("bf16", 50), ("f64", 120)])
def test_device_gmres_past_convergence(prec, iters):
    case("device gmres %s %d steps" % (prec, iters))
    qmg, lat, h, _ = _mg(24)
    r = random_spinors(DIMS, 3, 41)
    r[1] = 0.0
    taus = [0.02, 0.1, 2.5]
    prm = qmg.default_params(coarse_maxiter=iters, coarse_tol=0.0, nu_post=0, mg_prec=prec)
    z = host(lat.unpack(lat.vcycle(lat.field(3), lat.pack(dev(r)), taus, 3, prm), 3))
    assert not z[1].any()
    # P, the restricted right-hand side and the prolongated solution are rounded to the storage type
    tol = {"f64": 1e-13, "f32": 2.6e-5, "bf16": 3e-2}[prec]
    for k in (0, 2):
        assert _backward(h, mg.restrict(h.P, r[k], BLOCK), mg.restrict(h.P, z[k], BLOCK), taus[k]) < tol
