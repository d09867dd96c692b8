"""Stencil kernels for 4^4 blocks: every way the launch picks between them."""
import pytest

from gpu_common import case, dev, host, need_gpu
from helpers import oracle_at_sites, rel_err, sample_sites
from oracle import clover as oclover
from oracle import dirac
from synth import random_links, random_spinors, seed_for

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 16 blocks: few (one thread per site and direction) up to 8 rhs in FP64, 16 in FP32 and
# BF16; 32 blocks and more right-hand sides: a block per work-group, links held in FP32 and
# split over groups; tolerances of the FP64, FP32 and BF16 stencil
@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 1), ((8, 8, 8, 8), 9), ((8, 8, 8, 8), 17), ((4, 8, 16, 16), 17),
                                       ((4, 4, 4, 4), 3)])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 1e-6), ("bf16", 3e-2)])
@pytest.mark.parametrize("csw", [0.0, 1.0])
def test_stencil_selection(dims, nrhs, prec, tol, csw):
    case("stencil44 %s nrhs %d %s csw %g" % (dims, nrhs, prec, csw))
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    lat = qmg.Lattice(dims, (4, 4, 4, 4))
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


# 512 and 1024 blocks: one right-hand side without and with held links, outputs past 128 MB
@pytest.mark.parametrize("dims,nrhs,prec,tol", [((16, 16, 16, 32), 1, "f32", 1e-6), ((32, 16, 16, 32), 1, "f32", 1e-6),
                                                ((16, 16, 16, 32), 13, "f32", 1e-6), ((16, 16, 16, 32), 6, "f64", 1e-13)])
def test_stencil_selection_sampled(dims, nrhs, prec, tol):
    case("stencil44 sampled %s nrhs %d %s" % (dims, nrhs, prec))
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    lat = qmg.Lattice(dims, (4, 4, 4, 4))
    lat.set_gauge(dev(U), -0.8, 1.0)
    fin = lat.pack(dev(random_spinors(dims, nrhs, seed_for(2, "b"))), prec)
    pin = lat.unpack(fin, nrhs, prec)
    taus = [0.03 * (k + 1) for k in range(nrhs)]
    q = lat.unpack(lat.apply_Q_shifted(lat.field(nrhs, prec), fin, taus, nrhs, prec), nrhs, prec)
    sites = sample_sites(dims, 16, 4)
    for k in sorted({0, nrhs - 1}):
        ref = oracle_at_sites(U, host(pin[k]), -0.8, 1.0, sites, taus[k])
        assert rel_err([host(q[k][x]) for x in sites], ref) < tol


# a column alone and in batches that take other kernels: few-block kernel and the one that
# holds a block (8^4 and 16x8^3, FP64 from 9 and 5, FP32 and BF16 from 17 and 9 right-hand
# sides), links held or not (FP32), free and fixed order of loads on other blocks; bit for bit
@pytest.mark.parametrize("dims,block,batches", [((8, 8, 8, 8), (4, 4, 4, 4), (3, 9, 17)),
                                                ((16, 8, 8, 8), (4, 4, 4, 4), (5, 9, 12)),
                                                ((16, 16, 16, 8), (4, 4, 4, 4), (2, 5)),
                                                ((8, 8, 8, 8), (4, 4, 4, 2), (2, 17, 20)),
                                                ((16, 8, 8, 8), (8, 4, 4, 2), (2, 3))])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("csw", [0.0, 1.0])
def test_stencil_independent_of_batch(dims, block, batches, prec, csw):
    case("stencil batches %s %s %s csw %g" % (dims, block, prec, csw))
    qmg = need_gpu()
    lat = qmg.Lattice(dims, block)
    lat.set_gauge(dev(random_links(dims, 0.5, seed_for(2, "U"))), -0.8, csw)
    n = max(batches)
    fin, fb = lat.pack(dev(random_spinors(dims, n, seed_for(2, "b"))), prec), lat.field_bytes(prec)
    taus = [0.03 * (k + 1) for k in range(n)]
    for apply in (lat.apply_Q_shifted, lat.apply_A):
        ref = [apply(lat.field(1, prec), fin[k * fb:(k + 1) * fb], taus[k:k + 1], 1, prec) for k in range(n)]
        for m in batches:
            out = apply(lat.field(m, prec), fin[:m * fb], taus[:m], m, prec)
            for k in range(m):
                assert torch.equal(out[k * fb:(k + 1) * fb], ref[k]), (m, k)


def _pinned(lat, tmp_path, dims, order, variant):
    key = "gfx950|%s|4x4x4x4|clover=1" % "x".join(map(str, dims))
    entries = ['"%s|dslash|%s|%d": %d' % (key, p, c, variant) for p in ("f64", "f32", "bf16") for c in (0, 1)]
    path = tmp_path / ("tune_%d_%d.json" % (order, variant))
    path.write_text("{\n" + ",\n".join(entries + ['"%s|ds_order": %d' % (key, order)]) + "\n}\n")
    lat.autotune(str(path))


# work orders of the kernel that holds a block: 64 blocks (4x4x2x2, several tiles of every
# shape) and more right-hand sides than the few-block kernel takes, in FP32 in groups of one
# (5) and of three with a rest (17 in 6 groups), with today's variant number and old ones; the
# order changes which work-group computes what, so results are those of order 0 bit for bit
@pytest.mark.parametrize("prec,nrhs,tol", [("f64", 3, 1e-13), ("f32", 5, 1e-6), ("f32", 17, 1e-6), ("bf16", 5, 3e-2)])
@pytest.mark.parametrize("order,variant", [(1, 1), (3, 11), (5, 1), (7, 6)])
def test_stencil44_work_orders(order, variant, prec, nrhs, tol, tmp_path):
    case("stencil44 order %d variant %d %s nrhs %d" % (order, variant, prec, nrhs))
    qmg = need_gpu()
    dims = (16, 16, 8, 8)
    U = random_links(dims, 0.5, seed_for(2, "U"))
    lat = qmg.Lattice(dims, (4, 4, 4, 4))
    lat.set_gauge(dev(U), -0.8, 1.0)
    fin = lat.pack(dev(random_spinors(dims, nrhs, seed_for(2, "b"))), prec)
    taus = [0.03 * (k + 1) for k in range(nrhs)]
    _pinned(lat, tmp_path, dims, 0, 1)
    ref = lat.apply_Q_shifted(lat.field(nrhs, prec), fin, taus, nrhs, prec)
    _pinned(lat, tmp_path, dims, order, variant)
    out = lat.apply_Q_shifted(lat.field(nrhs, prec), fin, taus, nrhs, prec)
    assert torch.equal(out, ref)
    pin, q = host(lat.unpack(fin, nrhs, prec)), host(lat.unpack(out, nrhs, prec))
    sites = sample_sites(dims, 24, 4)
    for k in sorted({0, nrhs - 1}):
        want = oracle_at_sites(U, pin[k], -0.8, 1.0, sites, taus[k])
        assert rel_err([q[k][x] for x in sites], want) < tol


# the generic kernel on 4^4 blocks (variant 0) against the two 4^4 kernels on the same field
@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 2), ((16, 16, 8, 8), 5)])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 1e-6), ("bf16", 3e-2)])
def test_stencil44_generic(dims, nrhs, prec, tol, tmp_path):
    case("stencil44 generic %s %s nrhs %d" % (dims, prec, nrhs))
    qmg = need_gpu()
    lat = qmg.Lattice(dims, (4, 4, 4, 4))
    lat.set_gauge(dev(random_links(dims, 0.5, seed_for(2, "U"))), -0.8, 1.0)
    fin = lat.pack(dev(random_spinors(dims, nrhs, seed_for(2, "b"))), prec)
    taus = [0.03 * (k + 1) for k in range(nrhs)]
    got = []
    for variant in (0, 1):
        _pinned(lat, tmp_path, dims, 0, variant)
        got.append(host(lat.unpack(lat.apply_A(lat.field(nrhs, prec), fin, taus, nrhs, prec), nrhs, prec)))
    assert rel_err(got[0], got[1]) < tol
