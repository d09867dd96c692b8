"""Block shapes other than 4^4: SAP with slots of a wave, single waves, two and four waves per
block; the stencil with loads left free and in fixed order."""
import pytest

from gpu_common import case, dev, host, need_gpu
from helpers import rel_err
from oracle import clover as oclover
from oracle import dirac, sap
from synth import random_links, random_spinors, seed_for

pytestmark = pytest.mark.gpu


# blocks of 16 and 32 (four and two to a wave), 64, 128 and 256 sites; tolerances of the SAP
# on 4^4 blocks (same terms, other order)
@pytest.mark.parametrize("dims,block", [
    ((4, 8, 4, 4), (2, 2, 2, 2)), ((4, 4, 4, 8), (2, 2, 2, 4)), ((8, 4, 8, 4), (4, 2, 4, 2)),
    ((8, 8, 4, 8), (4, 4, 2, 4)), ((16, 8, 4, 8), (8, 4, 2, 4))])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 1e-6), ("bf16", 5e-2)])
@pytest.mark.parametrize("nrhs,csw", [(1, 0.0), (3, 1.0)])
def test_sap_block_shapes(dims, block, prec, tol, nrhs, csw):
    case("sap %s blocks %s %s nrhs %d" % (dims, block, prec, nrhs))
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(U), -0.8, csw)
    op = dirac.Operator(U, -0.8, oclover.clover_term(U, csw) if csw else None)
    f = random_spinors(dims, nrhs, seed_for(2, "b"))
    x0 = random_spinors(dims, nrhs, seed_for(2, "x"))
    taus = [0.02 * (k + 1) for k in range(nrhs)]
    fg, xg = lat.pack(dev(f), prec), lat.pack(dev(x0), prec)
    fin, xin = host(lat.unpack(fg, nrhs, prec)), host(lat.unpack(xg, nrhs, prec))
    got = host(lat.unpack(lat.sap_smooth(xg, fg, taus, nrhs, 2, 3, prec), nrhs, prec))
    for k in range(nrhs):
        assert rel_err(got[k], sap.sap(op, fin[k], xin[k], taus[k], block, 2, 3)) < tol


# few work-groups (free order), more than 256 of them and one right-hand side (both orders in
# FP32), blocks of 256 sites, a lattice smaller than a work-group; tolerances of the stencil
@pytest.mark.parametrize("dims,block,nrhs", [
    ((8, 8, 8, 8), (2, 2, 2, 2), 1), ((8, 8, 8, 8), (4, 4, 4, 2), 3), ((8, 8, 8, 8), (4, 2, 2, 4), 17),
    ((16, 4, 8, 4), (8, 4, 4, 2), 1), ((16, 4, 8, 4), (8, 4, 4, 2), 3), ((4, 4, 2, 4), (2, 2, 1, 4), 2)])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 1e-6), ("bf16", 3e-2)])
@pytest.mark.parametrize("csw", [0.0, 1.0])
def test_stencil_block_shapes(dims, block, nrhs, prec, tol, csw):
    case("stencil %s blocks %s nrhs %d %s csw %g" % (dims, block, nrhs, prec, csw))
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(U), -0.8, csw)
    C = oclover.clover_term(U, csw) if csw else None
    fin = lat.pack(dev(random_spinors(dims, nrhs, seed_for(2, "b"))), prec)
    pin = host(lat.unpack(fin, nrhs, prec))
    taus = [0.03 * (k + 1) for k in range(nrhs)]
    q = host(lat.unpack(lat.apply_Q_shifted(lat.field(nrhs, prec), fin, taus, nrhs, prec), nrhs, prec))
    a = host(lat.unpack(lat.apply_A(lat.field(nrhs, prec), fin, taus, nrhs, prec), nrhs, prec))
    for k in sorted({0, nrhs // 2, nrhs - 1}):
        assert rel_err(q[k], dirac.apply_Q_shifted(U, pin[k], -0.8, taus[k], C)) < tol
        assert rel_err(a[k], dirac.apply_A(U, pin[k], -0.8, taus[k], C)) < tol
