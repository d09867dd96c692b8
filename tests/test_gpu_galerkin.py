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
