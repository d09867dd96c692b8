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
