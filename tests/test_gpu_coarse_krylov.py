"""Coarse apply for few right-hand sides, device GMRES and dot products at their edges."""
import numpy as np
import pytest

from gpu_common import case, coarse_to_lex, dev, host, lex_to_coarse, need_gpu
from helpers import rel_err
from oracle import clover as oclover
from oracle import dirac, krylov, mg
from synth import random_links, random_spinors, random_test_vectors, seed_for

pytestmark = pytest.mark.gpu
DIMS, BLOCK = (8, 8, 8, 8), (4, 4, 4, 4)


def _mg(ntv):
    qmg = need_gpu()
    U = random_links(DIMS, 0.5, seed_for(2, "U"))
    op = dirac.Operator(U, -0.8, oclover.clover_term(U, 1.0))
    lat = qmg.Lattice(DIMS, BLOCK)
    lat.set_gauge(dev(U), -0.8, 1.0)
    W = random_test_vectors(DIMS, ntv, seed_for(2, "W"))
    lat.set_test_vectors(lat.pack(dev(W)), ntv)
    return qmg, lat, mg.TwoLevel(op, list(W), BLOCK), lat.coarse_site_order()


# one, two and up to four right-hand sides per work-group, row counts off the wave's 64 lanes
# and off the unrolling of 8; Q form: FP64 tolerance of the coarse apply
@pytest.mark.parametrize("ntv,nrhs", [(1, 1), (5, 1), (5, 3), (24, 2), (24, 3), (7, 6), (32, 1)])
def test_coarse_apply_few_rhs(ntv, nrhs):
    case("coarse apply ntv %d nrhs %d" % (ntv, nrhs))
    qmg, lat, h, order = _mg(ntv)
    rng = np.random.default_rng(8)
    y = rng.standard_normal((nrhs, len(order), 2 * ntv)) + 1j * rng.standard_normal((nrhs, len(order), 2 * ntv))
    taus = [0.02 * (k + 1) for k in range(nrhs)]
    og = lat.apply_coarse(lat.coarse(nrhs), dev(lex_to_coarse(y, order).view(np.float64)), taus, nrhs)
    out = coarse_to_lex(host(og).view(np.complex128), order, ntv)
    for k in range(nrhs):
        assert rel_err(out[k], h.coarse.apply(y[k], taus[k])) < 1e-13


# numbers of steps around the four basis vectors that a dot pass takes together; the V-cycle
# without smoothing returns the prolongated coarse solution; tolerance of the coarse GMRES
@pytest.mark.parametrize("iters", [1, 3, 4, 5, 9])
def test_device_gmres_steps(iters):
    case("device gmres %d steps" % iters)
    qmg, lat, h, order = _mg(8)
    r = random_spinors(DIMS, 3, 41)
    taus = [0.02, 0.1, -0.05]
    prm = qmg.default_params(coarse_maxiter=iters, coarse_tol=0.0, nu_post=0)
    z = host(lat.unpack(lat.vcycle(lat.field(3), lat.pack(dev(r)), taus, 3, prm), 3))
    for k in range(3):
        y, _, _ = krylov.gmres(lambda v: h.coarse.apply(v, taus[k]), mg.restrict(h.P, r[k], BLOCK), iters)
        assert rel_err(z[k], mg.prolong(h.P, y, DIMS, BLOCK)) < 1e-13


# 3072 and 12288 entries: chunks of 2048 with and without a remainder; the sums run in FP64
# over the stored values, so 1e-12 of the value holds for every storage type
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (4, 4, 8, 8)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_field_dot_remainder(dims, prec):
    case("field dot %s %s" % (dims, prec))
    qmg = need_gpu()
    lat = qmg.Lattice(dims, (2, 2, 2, 2))
    a, b = (lat.pack(dev(random_spinors(dims, 3, s)), prec) for s in (5, 6))
    av, bv = host(lat.unpack(a, 3, prec)), host(lat.unpack(b, 3, prec))
    got = lat.field_dot(a, b, 3, prec)
    for k in range(3):
        scale = np.linalg.norm(av[k]) * np.linalg.norm(bv[k])
        assert abs(got[k] - np.vdot(av[k], bv[k])) < 1e-12 * scale


# matrix-core apply: 2 ntv in one, two and three tiles of 16 rows, both packings (up to 8 and
# up to 16 right-hand sides) at their edges, 256 sites where one and two right-hand sides take
# it too; rel. 1e-13 (FP64: sums of 9 * 48 products),
# 9 * 48 * 2^-24 = 2.6e-5 (FP32: rounding of blocks, inputs and every partial sum)
@pytest.mark.parametrize("dims,block,ntv,nrhs", [
    ((8, 8, 8, 8), (4, 4, 4, 4), 8, 3), ((8, 8, 8, 8), (4, 4, 4, 4), 16, 8), ((8, 8, 8, 8), (4, 4, 4, 4), 24, 9),
    ((8, 8, 8, 8), (4, 4, 4, 4), 24, 16), ((8, 8, 8, 8), (4, 4, 4, 4), 16, 17), ((8, 8, 8, 8), (2, 2, 2, 2), 24, 1),
    ((8, 8, 8, 8), (2, 2, 2, 2), 24, 2)])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 2.6e-5)])
def test_coarse_apply_matrix_cores(dims, block, ntv, nrhs, prec, tol):
    case("coarse apply %s ntv %d nrhs %d %s" % (dims, ntv, nrhs, prec))
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    op = dirac.Operator(U, -0.8, oclover.clover_term(U, 1.0))
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(U), -0.8, 1.0)
    W = random_test_vectors(dims, ntv, seed_for(2, "W"))
    lat.set_test_vectors(lat.pack(dev(W)), ntv)
    h, order = mg.TwoLevel(op, list(W), block), lat.coarse_site_order()
    rng = np.random.default_rng(8)
    y = rng.standard_normal((nrhs, len(order), 2 * ntv)) + 1j * rng.standard_normal((nrhs, len(order), 2 * ntv))
    taus = [0.02 * (k + 1) for k in range(nrhs)]
    real = np.float64 if prec == "f64" else np.float32
    yd = dev(lex_to_coarse(y, order).view(np.float64).astype(real))
    og = lat.apply_coarse(lat.coarse(nrhs, prec), yd, taus, nrhs, prec)
    out = coarse_to_lex(host(og).view(real).astype(np.float64).view(np.complex128), order, ntv)
    for k in range(nrhs):
        assert rel_err(out[k], h.coarse.apply(y[k], taus[k])) < tol


# one wave per site: 512 and 1024 sites, where it takes over from nine (FP64: 1, 2, 4 and 8 right-hand
# sides, 3 of them one at a time; FP32: 3 and 8), and rows longer than half a wave; Q form by
# the V-cycle tests.  rel. 1e-13 and 2.6e-5 as above
@pytest.mark.parametrize("dims,ntv,nrhs", [((8, 8, 8, 16), 5, 4), ((8, 8, 8, 16), 5, 8), ((8, 8, 16, 16), 12, 1),
                                           ((8, 8, 16, 16), 12, 2), ((8, 8, 16, 16), 12, 3), ((8, 8, 16, 16), 5, 9),
                                           ((8, 8, 16, 16), 20, 3), ((8, 8, 16, 16), 28, 3)])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 2.6e-5)])
def test_coarse_apply_many_sites(dims, ntv, nrhs, prec, tol):
    case("coarse apply many sites %s ntv %d nrhs %d %s" % (dims, ntv, nrhs, prec))
    qmg = need_gpu()
    block = (2, 2, 2, 2)
    U = random_links(dims, 0.5, seed_for(2, "U"))
    op = dirac.Operator(U, -0.8, None)
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(U), -0.8, 0.0)
    W = random_test_vectors(dims, ntv, seed_for(2, "W"))
    lat.set_test_vectors(lat.pack(dev(W)), ntv)
    P, order = mg.build_P(W, block), lat.coarse_site_order()
    rng = np.random.default_rng(8)
    y = rng.standard_normal((nrhs, len(order), 2 * ntv)) + 1j * rng.standard_normal((nrhs, len(order), 2 * ntv))
    taus = [0.02 * (k + 1) for k in range(nrhs)]
    real = np.float64 if prec == "f64" else np.float32
    yd = dev(lex_to_coarse(y, order).view(np.float64).astype(real))
    og = lat.apply_coarse(lat.coarse(nrhs, prec), yd, taus, nrhs, prec)
    out = coarse_to_lex(host(og).view(real).astype(np.float64).view(np.complex128), order, ntv)
    for k in sorted({0, nrhs - 1}):
        assert rel_err(out[k], mg.restrict(P, op.A(mg.prolong(P, y[k], dims, block), taus[k]), block)) < tol
