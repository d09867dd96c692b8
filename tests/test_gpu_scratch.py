"""The smoother's halo field when device memory is short."""
import pytest

from gpu_common import case, dev, host, need_gpu
from helpers import rel_err
from synth import random_links, random_spinors, random_test_vectors, seed_for

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DIMS, NRHS, NTV = (16, 16, 16, 32), 64, 8
LEAVE = 256 << 20  # left free; the halo of 64 FP32 right-hand sides takes 805 MB


def _lat(tmp_path, sap):
    qmg = need_gpu()
    lat = qmg.Lattice(DIMS, (4, 4, 4, 4))
    lat.set_gauge(dev(random_links(DIMS, 0.5, seed_for(2, "U"))), -0.8, 1.0)
    lat.set_test_vectors(lat.pack(dev(random_test_vectors(DIMS, NTV, seed_for(2, "W")))), NTV)
    _pin(lat, tmp_path, sap)
    return qmg, lat


def _pin(lat, tmp_path, sap):
    key = "gfx950|%s|4x4x4x4|clover=1" % "x".join(map(str, DIMS))
    entries = ['"%s|dslash|%s|%d": 1' % (key, p, c) for p in ("f64", "f32", "bf16") for c in (0, 1)]
    path = tmp_path / ("tune_%d.json" % sap)
    path.write_text("{\n" + ",\n".join(entries + ['"%s|sap": %d' % (key, sap)]) + "\n}\n")
    lat.autotune(str(path))


def _fill():
    """Takes all device memory but LEAVE, in pieces until there is no more (the memory is not touched)."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held, size = [], 32 << 30
    while size >= 32 << 20:
        try:
            held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            size //= 2
    given = 0
    while given < LEAVE:
        given += held.pop().numel()
    torch.cuda.empty_cache()
    if given > LEAVE:
        held.append(torch.empty(given - LEAVE, dtype=torch.uint8, device="cuda"))
    print("held %d pieces, %.1f GB, %d MB free" % (len(held), sum(h.numel() for h in held) / 1e9,
                                                  torch.cuda.mem_get_info()[0] >> 20), flush=True)
    return held


def test_graph_vcycle_without_room_for_the_halo(tmp_path):
    """The eager run finds no room and gathers; the recorded one has to do the same instead of
    allocating under the capture.  FP32 tolerance of V-cycles against the result with a halo."""
    case("graph V-cycle without room for the halo")
    qmg, lat = _lat(tmp_path, 1)  # gathering kernels: every other buffer gets its size
    r = lat.pack(dev(random_spinors(DIMS, 4, 41))).repeat(NRHS // 4)
    taus = [0.01 * (k % 7) for k in range(NRHS)]
    prm = qmg.default_params(mg_prec="f32", use_graph=1, coarse_maxiter=4)
    z = lat.field(NRHS)
    lat.vcycle(z, r, taus, NRHS, prm)
    _pin(lat, tmp_path, 2)
    full = _fill()
    try:
        for _ in range(3):
            z.zero_()
            lat.vcycle(z, r, taus, NRHS, prm)
    finally:
        del full
        torch.cuda.empty_cache()
    short = z.clone()
    _pin(lat, tmp_path, 2)  # drops the recorded V-cycle
    lat.vcycle(z, r, taus, NRHS, prm)
    for k in (0, 5, NRHS - 1):
        one = slice(k * lat.field_bytes(), (k + 1) * lat.field_bytes())
        assert rel_err(host(lat.unpack(short[one])), host(lat.unpack(z[one]))) < 1e-6


def test_halo_given_back(tmp_path):
    """A later call that needs its memory gets it; the smoother goes on without, and with it
    again once there is room."""
    case("halo given back")
    _, lat = _lat(tmp_path, 2)
    f, x = lat.pack(dev(random_spinors(DIMS, 4, 41)), "f32").repeat(NRHS // 4), lat.field(NRHS, "f32")
    taus = [0.01 * (k % 7) for k in range(NRHS)]
    ref = lat.sap_smooth(x.clone(), f, taus, NRHS, 2, 2, "f32").clone()  # allocates the halo
    y, yo = lat.coarse(NRHS, "f32"), lat.coarse(NRHS, "f32")
    y.view(torch.float32).normal_()
    x2 = x.clone()
    full = _fill()
    try:
        # a basis of 121 vectors of 64 x 512 x 16 complex entries: 508 MB
        lat.coarse_solve(yo, y, taus, NRHS, 120, 1e-4, "f32")
        lat.sap_smooth(x2, f, taus, NRHS, 2, 2, "f32")
        torch.cuda.synchronize()
    finally:
        del full
        torch.cuda.empty_cache()
    assert rel_err(x2.view(torch.float32).cpu(), ref.view(torch.float32).cpu()) < 1e-6
    assert torch.equal(lat.sap_smooth(x, f, taus, NRHS, 2, 2, "f32"), ref)
