"""Packing, link packing and the gauge force where lattices do not fill the tiles."""
import numpy as np
import pytest

from gpu_common import case, dev, host, need_gpu
from helpers import rel_err
from oracle import dirac, force
from synth import random_links, random_spinors, seed_for

pytestmark = pytest.mark.gpu


# fewer sites than a tile of 64 or 256, remainders of both, blocks smaller and larger than a
# tile; FP64 tolerance of the stencil and the force
@pytest.mark.parametrize("dims,block", [((2, 2, 2, 4), (2, 2, 2, 2)), ((6, 2, 2, 2), (2, 2, 2, 2)),
                                        ((4, 6, 4, 4), (4, 2, 2, 1)), ((8, 8, 4, 8), (8, 8, 4, 4)),
                                        ((4, 4, 4, 12), (4, 4, 4, 4))])
def test_tiles(dims, block):
    case("layout %s %s" % (dims, block))
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    psi = random_spinors(dims, 3, seed_for(2, "b"))
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(U), -0.8, 0.0)
    f = lat.pack(dev(psi))
    assert np.array_equal(host(lat.unpack(f, 3)), psi)
    for prec, cast in (("f32", np.complex64), ("bf16", None)):
        g = host(lat.unpack(lat.pack(dev(psi), prec), 3, prec))
        assert rel_err(g, psi) < (1e-7 if cast else 4e-3)
        if cast:
            assert np.array_equal(g, psi.astype(cast).astype(np.complex128))
    for prec, tol in (("f64", 1e-13), ("f32", 1e-6), ("bf16", 3e-2)):
        g = lat.pack(dev(psi), prec)
        q = host(lat.unpack(lat.apply_Q(lat.field(3, prec), g, 3, prec), 3, prec))
        p = host(lat.unpack(g, 3, prec))
        assert rel_err(q[2], dirac.apply_Q(U, p[2], -0.8)) < tol
    fb = lat.field_bytes()
    G, Gb = (host(t) for t in lat.gauge_force(f[:fb], f[fb:2 * fb]))
    ref = force.gauge_force(psi[0], psi[1])
    assert rel_err(G, ref[0]) < 1e-13 and rel_err(Gb, ref[1]) < 1e-13
