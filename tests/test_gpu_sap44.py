"""SAP on 4^4 blocks with the halo field between half-sweeps."""
import numpy as np
import pytest

from gpu_common import case, dev, host, need_gpu
from helpers import rel_err
from oracle import clover as oclover
from oracle import dirac, sap
from synth import random_links, random_spinors, seed_for

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BLOCK = (4, 4, 4, 4)


def _lat(dims, csw, m0=-0.8):
    qmg = need_gpu()
    U = random_links(dims, 0.5, seed_for(2, "U"))
    lat = qmg.Lattice(dims, BLOCK)
    lat.set_gauge(dev(U), m0, csw)
    return lat, dirac.Operator(U, m0, oclover.clover_term(U, csw) if csw else None)


# both neighbours of a block the same block (two per direction) and not; one, an odd number
# and more right-hand sides than work-groups take at a time; one sweep (no halo after it) and
# more; tolerances as for the kernels that gather the neighbours (same terms, other order)
@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (16, 8, 8, 16)])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-13), ("f32", 1e-6), ("bf16", 5e-2)])
@pytest.mark.parametrize("nrhs,csw,nsweep,n_mr", [(1, 1.0, 1, 2), (3, 0.0, 3, 3), (17, 1.0, 2, 3)])
def test_sap_halo(dims, prec, tol, nrhs, csw, nsweep, n_mr):
    case("sap44 %s %s nrhs %d csw %g" % (dims, prec, nrhs, csw))
    lat, op = _lat(dims, csw)
    f = random_spinors(dims, nrhs, seed_for(2, "b"))
    x0 = random_spinors(dims, nrhs, seed_for(2, "x"))
    taus = [0.02 * (k + 1) for k in range(nrhs)]
    fg, xg = lat.pack(dev(f), prec), lat.pack(dev(x0), prec)
    fin, xin = host(lat.unpack(fg, nrhs, prec)), host(lat.unpack(xg, nrhs, prec))
    got = host(lat.unpack(lat.sap_smooth(xg, fg, taus, nrhs, nsweep, n_mr, prec), nrhs, prec))
    for k in sorted({0, nrhs - 1}):
        assert rel_err(got[k], sap.sap(op, fin[k], xin[k], taus[k], BLOCK, nsweep, n_mr)) < tol


def test_sap_halo_streams_and_capture():
    """Calls in flight on two streams at a time share the halo field in turn; a caller's
    own capture takes the kernels that need no scratch."""
    case("sap44 streams, capture")
    dims, nrhs = (16, 8, 8, 8), 3
    lat, _ = _lat(dims, 1.0)
    f = [lat.pack(dev(random_spinors(dims, nrhs, 100 + i)), "f32") for i in range(2)]
    x0 = lat.pack(dev(random_spinors(dims, nrhs, 7)), "f32")
    taus = [0.01, 0.02, 0.03]
    ref = [lat.sap_smooth(x0.clone(), f[i], taus, nrhs, 3, 3, "f32").clone() for i in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    xs = [[x0.clone() for _ in range(8)] for _ in range(2)]
    torch.cuda.synchronize()
    for j in range(8):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                lat.sap_smooth(xs[i][j], f[i], taus, nrhs, 3, 3, "f32")
    torch.cuda.synchronize()
    for i in range(2):
        for j in range(8):
            assert torch.equal(xs[i][j], ref[i])
    xc = x0.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lat.sap_smooth(xc, f[0], taus, nrhs, 3, 3, "f32")
    for _ in range(3):
        xc.copy_(x0)
        g.replay()
        torch.cuda.synchronize()
        a, b = xc.view(torch.float32).double(), ref[0].view(torch.float32).double()
        assert float((a - b).abs().max() / b.abs().max()) < 1e-6


def test_sap_halo_groups():
    """48 right-hand sides of 64x32^3 need more halo than is kept and go in two groups:
    each column equals the column smoothed alone, bit for bit."""
    case("sap44 groups 64x32^3 48 rhs")
    qmg = need_gpu()
    dims, nrhs = (64, 32, 32, 32), 48
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    lat = qmg.Lattice(dims, BLOCK)
    U = 0.4 * torch.view_as_complex(torch.randn(dims + (4, 3, 3, 2), generator=g, device="cuda", dtype=torch.float64))
    lat.set_gauge(U, 0.5, 0.0)
    del U
    fb = lat.field_bytes("f32")
    f = torch.randn(nrhs * fb // 4, generator=g, device="cuda", dtype=torch.float32).view(torch.uint8)
    x = lat.field(nrhs, "f32")
    taus = [0.001 * k for k in range(nrhs)]
    lat.sap_smooth(x, f, taus, nrhs, 2, 2, "f32")
    for k in (0, 41, 42, 47):
        y = lat.field(1, "f32")
        lat.sap_smooth(y, f[k * fb:(k + 1) * fb], [taus[k]], 1, 2, 2, "f32")
        assert torch.equal(y, x[k * fb:(k + 1) * fb]), k
