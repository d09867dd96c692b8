"""P and D_c built from test vectors: panels, tiles and faces at their edges."""
import numpy as np
import pytest

from gpu_common import case, dev, host, need_gpu
from helpers import rel_err
from oracle import clover as oclover
from oracle import dirac, mg
from synth import random_links, random_spinors, random_test_vectors, seed_for

pytestmark = pytest.mark.gpu


# numbers of vectors around the six columns of a panel and the 16 of a tile; blocks with
# fewer sites than a wave, faces that are not a multiple of the 16 sites taken at a time;
# tolerance as for the FP64 coarse apply and transfers
@pytest.mark.parametrize("dims,block,ntv,csw", [((8, 8, 8, 8), (4, 4, 4, 4), 1, 1.0), ((8, 8, 8, 8), (4, 4, 4, 4), 7, 0.0),
                                                ((8, 8, 8, 8), (4, 4, 4, 4), 17, 1.0),
                                                ((8, 8, 8, 16), (4, 4, 4, 4), 32, 1.0),
                                                ((8, 8, 4, 4), (4, 4, 2, 2), 12, 1.0),
                                                ((4, 4, 4, 16), (2, 2, 2, 8), 6, 1.0),
                                                ((4, 4, 4, 4), (2, 2, 2, 2), 24, 1.0)])
def test_interpolation_and_coarse_operator(dims, block, ntv, csw):
    case("galerkin %s %s ntv %d" % (dims, block, ntv))
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    op = dirac.Operator(U, -0.8, oclover.clover_term(U, csw) if csw else None)
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(U), -0.8, csw)
    W = random_test_vectors(dims, ntv, seed_for(2, "W"))
    lat.set_test_vectors(lat.pack(dev(W)), ntv)
    P = mg.build_P(W, block)
    order = np.array(lat.coarse_site_order())
    nb = len(order)
    rng = np.random.default_rng(5)
    y = rng.standard_normal((nb, 2 * ntv)) + 1j * rng.standard_normal((nb, 2 * ntv))
    yg = dev(y[order])
    v = host(lat.unpack(lat.prolong(lat.field(1), yg, 1)))[0]
    ref = mg.prolong(P, y, dims, block)
    assert rel_err(v, ref) < 1e-13
    out = lat.apply_coarse(lat.coarse(1), yg, [0.03], 1)
    got = host(out).view(np.complex128).reshape(nb, 2 * ntv)
    want = mg.restrict(P, op.A(ref, 0.03), block)
    assert rel_err(got, want[order]) < 1e-13
    # the reduced-precision copies hold the same P
    b = random_spinors(dims, 1, seed_for(2, "b"))
    for prec, tol in (("f32", 2e-6), ("bf16", 3e-2)):
        r = lat.restrict(lat.coarse(1, prec), lat.pack(dev(b), prec), 1, prec)
        r = host(r).view(np.complex64).reshape(nb, 2 * ntv)
        assert rel_err(r, mg.restrict(P, b[0], block)[order]) < tol


# six and more vectors that agree to 1e-9 .. 1e-11, within and across the panels: P's columns
# stay orthonormal to the tolerance of the FP64 transfers (P^H P y = y), and the difference of
# two vectors lies in its range up to the rounding of 2 ntv subtractions of vectors 1 / eps
# times as large (twice that: maxima against norms)
@pytest.mark.parametrize("ntv,eps", [(4, 1e-9), (6, 1e-10), (6, 1e-11), (13, 1e-10), (24, 1e-11)])
def test_interpolation_of_close_vectors(ntv, eps):
    case("galerkin close vectors ntv %d eps %g" % (ntv, eps))
    qmg = need_gpu()
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(random_links(dims, 0.5, seed_for(2, "U"))), -0.8, 0.0)
    d = random_spinors(dims, ntv + 1, 17)
    W = d[0][None] + eps * d[1:]
    lat.set_test_vectors(lat.pack(dev(W)), ntv)
    rng = np.random.default_rng(6)
    y = rng.standard_normal((16, 2 * ntv)) + 1j * rng.standard_normal((16, 2 * ntv))
    v = lat.prolong(lat.field(1), dev(y), 1)
    got = host(lat.restrict(lat.coarse(1), v, 1)).view(np.complex128).reshape(y.shape)
    assert rel_err(got, y) < 1e-13
    w = lat.pack(dev(W[-1] - W[0]))
    pw = host(lat.unpack(lat.prolong(lat.field(1), lat.restrict(lat.coarse(1), w, 1), 1)))[0]
    assert rel_err(pw, W[-1] - W[0]) < 4 * ntv * 1.1e-16 / eps
