"""Gradient smoothing (Laplace and Bessel filters) on the GPU against the
FP64 oracle (oracle/smooth.py) on a ragged volume, plus its use in the FWI
gradient."""

import numpy as np
import pytest

from oracle import smooth as osm
from gpu_util import gpu_or_skip, rel_l2, say

pytestmark = pytest.mark.gpu

SHAPE = (11, 17, 23)   # [z][y][x]
H = (10.0, 12.0, 8.0)  # (x, y, z)


@pytest.mark.parametrize("mode", ["laplace", "bessel"])
def test_smoothing_matches_oracle(mode):
    torch = gpu_or_skip()
    from paper_2502_12350_amd import smooth
    rng = np.random.default_rng(7)
    g = rng.standard_normal(SHAPE).astype(np.float32)
    lens = (2 * H[0], 3 * H[1], 1.5 * H[2])
    ref = (osm.laplace_filter if mode == "laplace" else osm.bessel_filter)(g, lens, H)
    out, it = smooth(torch.from_numpy(g).cuda(), mode, lens, H, tol=1e-7)
    torch.cuda.synchronize()
    e = rel_l2(out.cpu().numpy(), ref)
    say(f"[smooth {mode}] rel-L2 {e:.2e}, {it} iterations")
    assert e <= 1e-5
    # constants are kept
    c, _ = smooth(torch.full(SHAPE, 2.5, device="cuda"), mode, lens, H, tol=1e-7)
    assert float((c - 2.5).abs().max()) <= 1e-5
    if mode == "laplace":  # in place gives the same bits
        x = torch.from_numpy(g).cuda()
        smooth(x, mode, lens, H, out=x)
        assert torch.equal(x, out)


def test_smoothing_errors():
    torch = gpu_or_skip()
    from paper_2502_12350_amd import smooth, WfdError
    x = torch.zeros(SHAPE, device="cuda")
    with pytest.raises(WfdError):
        smooth(x, "bessel", (10.0, 10.0, 10.0), H, out=x)       # needs out != in
    with pytest.raises(WfdError):
        smooth(x, "laplace", (-1.0, 10.0, 10.0), H)
    with pytest.raises(WfdError) as e:                          # too few iterations
        smooth(torch.randn(SHAPE, device="cuda"), "bessel", (40.0, 40.0, 40.0), H,
               tol=1e-9, max_iter=2)
    assert e.value.name == "WFD_E_RANGE"


def test_fwi_gradient_smoothing_is_applied_before_zeroing():
    torch = gpu_or_skip()
    import seisgen
    from paper_2502_12350_amd import GridSpec, Propagator, smooth
    from paper_2502_12350_amd.fwi import Shots, evaluate
    w = seisgen.workload("c4_fd")
    g = GridSpec(**w.grid_kwargs())
    P = Propagator(0)
    P.set_model(g, torch.from_numpy(w.vel + 5.0 * w.extra["dv"]).cuda())
    wav = torch.from_numpy(w.wavelet).cuda()
    d = P.forward(wav, w.sources[0], w.receivers).clone()
    shots = Shots(wav, np.asarray(w.sources), [w.receivers], [d])
    v = torch.from_numpy(w.vel).cuda()
    _, raw = evaluate(P, g, v, None, shots, ckpt="full")
    raw = raw.clone()
    lens = (20.0, 20.0, 20.0)
    _, sm = evaluate(P, g, v, None, shots, ckpt="full", zero_top_planes=3,
                     smoothing=("bessel", lens))
    ref, _ = smooth(raw, "bessel", lens, (w.dx, w.dy, w.dz))
    ref[:3] = 0.0
    torch.cuda.synchronize()
    assert float((sm - ref).abs().max()) <= 1e-6 * float(ref.abs().max())


@pytest.mark.parametrize("mode", ["nearest", "sinc"])
def test_resampling_matches_oracle(mode):
    torch = gpu_or_skip()
    from oracle import resample as ors
    from paper_2502_12350_amd import resample
    rng = np.random.default_rng(9)
    d = rng.standard_normal((37, 300)).astype(np.float32)
    for dt_in, nt_out, dt_out in ((2e-3, 600, 1e-3), (1e-3, 130, 2.3e-3), (1.5e-3, 300, 1.5e-3)):
        ref = ors.resample(d, dt_in, nt_out, dt_out, mode)
        got = resample(torch.from_numpy(d).cuda(), dt_in, nt_out, dt_out, mode)
        torch.cuda.synchronize()
        g = got.cpu().numpy().astype(np.float64)
        if mode == "nearest":
            assert np.array_equal(g, ref)
        else:
            e = rel_l2(g, ref)
            say(f"[resample sinc] dt {dt_in} -> {dt_out}: rel-L2 {e:.2e}")
            assert e <= 1e-6


@pytest.mark.parametrize("nrec, nt_in, nt_out", [
    (1, 1, 1), (1, 15, 64), (16, 16, 16), (17, 17, 65), (33, 31, 63), (70, 64, 129),
    (129, 47, 300), (700, 33, 1100)])
def test_sinc_resampling_tiles(nrec, nt_in, nt_out):
    """Around the 16-sample and 16-trace tiles and every number of row tiles.
    FP64 sums rounded once to FP32: at most 2^-24 of each value."""
    torch = gpu_or_skip()
    from oracle import resample as ors
    from paper_2502_12350_amd import resample
    d = np.random.default_rng(nrec).standard_normal((nrec, nt_in)).astype(np.float32)
    for dt_out in (0.5e-3, 0.7e-3, 1.9e-3):   # on samples every second time, and never
        ref = ors.resample(d, 1.0e-3, nt_out, dt_out, "sinc")
        got = resample(torch.from_numpy(d).cuda(), 1.0e-3, nt_out, dt_out, "sinc")
        assert rel_l2(got.cpu().numpy(), ref) <= 1e-7


@pytest.mark.parametrize("shape", [
    (1, 1, 1), (2, 3, 1), (5, 65, 64), (33, 130, 257), (3, 5, 1900), (2050, 3, 33), (2, 700, 40),
    (1, 1, 4000), (1, 9000, 2)])
def test_laplace_tiles(shape):
    """Line tiles of every size, ragged ones, and lines too long for a tile.
    Each axis rounds twice to FP32 (2^-24 relative to the line's largest
    value), six roundings in all."""
    torch = gpu_or_skip()
    from paper_2502_12350_amd import smooth
    g = np.random.default_rng(3).standard_normal(shape).astype(np.float32)
    for lens in ((20.0, 30.0, 12.0), (500.0, 0.0, 1.0)):
        ref = osm.laplace_filter(g, lens, H)
        x = torch.from_numpy(g).cuda()
        out, _ = smooth(x, "laplace", lens, H)
        tol = 6 * 2.0 ** -24 * max(1.0, float(np.abs(g).max()))
        assert float(np.abs(out.cpu().numpy() - ref).max()) <= tol
        smooth(x, "laplace", lens, H, out=x)
        assert torch.equal(x, out)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 2, 300), (70, 3, 2), (9, 33, 31), (3, 16, 16),
                                   (40, 17, 15)])
def test_bessel_blocks(shape):
    """Planes below, at and above a block's 256 points, and ends on every axis.
    The residual tolerance bounds the error relative to the input (B >= I);
    every iteration adds a few roundings of 2^-24."""
    torch = gpu_or_skip()
    from paper_2502_12350_amd import smooth
    g = np.random.default_rng(5).standard_normal(shape).astype(np.float32)
    for lens in ((20.0, 30.0, 12.0), (60.0, 0.0, 40.0)):
        ref = osm.bessel_filter(g, lens, H)
        out, it = smooth(torch.from_numpy(g).cuda(), "bessel", lens, H, tol=1e-7)
        assert it >= 1
        assert np.linalg.norm(out.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(g)
    out, it = smooth(torch.zeros(shape, device="cuda"), "bessel", lens, H)
    assert it == 0 and float(out.abs().max()) == 0.0


@pytest.mark.parametrize("dt_in, dt_out, nt_in, nt_out", [
    (1.0e-3, 0.7e-3, 9000, 12600), (4.0e-3, 1.6e-3, 8600, 21300)])
def test_sinc_resampling_far_along_a_trace(dt_in, dt_out, nt_in, nt_out):
    """Positions past 8192 samples that miss their sample by a rounding of the
    position (more than the 1e-12 within which a position counts as on it).
    FP64 sums rounded once to FP32: 2^-24 of each value; the oracle's and the
    kernel's positions differ by a few 1e-12 samples, which moves a value by
    less than 1e-10 of the largest."""
    torch = gpu_or_skip()
    from oracle import resample as ors
    from paper_2502_12350_amd import resample
    d = np.random.default_rng(11).standard_normal((2, nt_in)).astype(np.float32)
    ref = ors.resample(d, dt_in, nt_out, dt_out, "sinc")
    got = resample(torch.from_numpy(d).cuda(), dt_in, nt_out, dt_out, "sinc").cpu().numpy()
    err = np.abs(got - ref) - 2.0 ** -24 * np.abs(ref)
    assert float(err.max()) <= 1e-9 * float(np.abs(d).max())


@pytest.mark.parametrize("shape, axis", [
    ((901, 190, 211), 2), ((30, 1100, 1500), 1), ((1402, 199, 251), 2), ((70, 31, 1399), 0)])
def test_laplace_marched_lines(shape, axis):
    """Lines marched in memory: copied first (a volume in the last-level cache, x
    lines) or from the input, and in place.  Two FP32 roundings along the axis."""
    torch = gpu_or_skip()
    from paper_2502_12350_amd import smooth
    g = np.random.default_rng(13).standard_normal(shape).astype(np.float32)
    lens = [0.0, 0.0, 0.0]
    lens[axis] = 30.0
    ref = osm.laplace_filter(g, lens, H)
    x = torch.from_numpy(g).cuda()
    out, _ = smooth(x, "laplace", lens, H)
    assert float(np.abs(out.cpu().numpy() - ref).max()) <= 2 * 2.0 ** -24 * float(np.abs(g).max())
    smooth(x, "laplace", lens, H, out=x)
    assert torch.equal(x, out)


def _bessel_by_cosines(g, lens):
    """B^-1 g in FP64 by the cosine bases that diagonalise the zero-flux second
    differences (equal to the oracle's direct solve where that is feasible)."""
    from scipy.fft import dctn, idctn
    lam = 1.0
    for axis in range(3):
        n, l, h = g.shape[axis], lens[2 - axis], H[2 - axis]
        e = (l / h) ** 2 * (2.0 - 2.0 * np.cos(np.pi * np.arange(n) / n))
        lam = lam + e.reshape([n if a == axis else 1 for a in range(3)])
    return idctn(dctn(g.astype(np.float64)) / lam)


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (40, 90, 70), (3, 730, 731),
                                   (30, 200, 210)])
def test_bessel_with_the_least_workspace(shape):
    """Three volumes and the published 4096 bytes: fewer blocks, that take several
    items each where there are more than 252 (and, with the full workspace, in
    planes of more than 2048 blocks of 256 points).  Tolerance as above."""
    torch = gpu_or_skip()
    import ctypes as C
    from paper_2502_12350_amd import _lib, smooth
    from paper_2502_12350_amd.api import _dptr
    g = np.random.default_rng(5).standard_normal(shape).astype(np.float32)
    nz, ny, nx = shape
    x = torch.from_numpy(g).cuda()
    lens, h = np.array([20.0, 30.0, 12.0]), np.ascontiguousarray(H, dtype=np.float64)
    ref = _bessel_by_cosines(g, lens)
    if g.size < 200:
        assert np.allclose(ref, osm.bessel_filter(g, lens, H), rtol=0, atol=1e-12)
    nbytes = (12 * g.size + 255) // 256 * 256 + 4096
    n = C.c_size_t()
    _lib.check(_lib.lib().wfd_smooth_workspace_bytes(_lib.SMOOTH_BESSEL, nx, ny, nz, C.byref(n)))
    assert n.value <= nbytes
    out, it = torch.empty_like(x), C.c_int32()
    # canaries on either side
    buf = torch.full((nbytes + 2 * 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    _lib.check(_lib.lib().wfd_smooth(_lib.SMOOTH_BESSEL, x.data_ptr(), out.data_ptr(), nx, ny, nz,
                                     _dptr(lens), _dptr(h), 1e-7, 500, buf.data_ptr() + 4096,
                                     nbytes, C.byref(it), None))
    assert it.value >= 1
    assert np.linalg.norm(out.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(g)
    assert bool((buf[:4096] == 0x5a).all()) and bool((buf[4096 + nbytes:] == 0x5a).all())
    full, it_full = smooth(x, "bessel", lens, H, tol=1e-7)
    assert it_full == it.value
    assert np.linalg.norm(full.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(g)


@pytest.mark.parametrize("nrec, nt_in, nt_out", [
    (2100, 40, 1030),         # four row tiles a wavefront
    (1300, 50, 700),          # two
    (67_200_000, 1, 1)])      # more row blocks than a launch takes: rows in turn
def test_sinc_resampling_row_tiles(nrec, nt_in, nt_out):
    """As test_sinc_resampling_tiles, at sizes that take several row tiles; the
    last one's single weight is sinc(dt_out / dt_in - 1)."""
    torch = gpu_or_skip()
    from oracle import resample as ors
    from paper_2502_12350_amd import resample
    rng = torch.Generator(device="cuda").manual_seed(nrec)
    d = torch.randn((nrec, nt_in), generator=rng, device="cuda")
    dt_out = 0.7e-3
    got = resample(d, 1.0e-3, nt_out, dt_out, "sinc")
    if nt_in > 1:
        ref = ors.resample(d.cpu().numpy(), 1.0e-3, nt_out, dt_out, "sinc")
        assert rel_l2(got.cpu().numpy(), ref) <= 1e-7
    else:
        ref = d.double() * float(np.sinc(dt_out / 1.0e-3 - 1.0))
        assert float(((got - ref).abs() - 2.0 ** -24 * ref.abs()).max()) <= 1e-14


@pytest.mark.parametrize("nrec, nt_in, nt_out", [(1, 1, 1), (3, 7, 85), (5, 300, 256), (700, 33, 257)])
def test_nearest_resampling_edges(nrec, nt_in, nt_out):
    """Below, at and above a block of 256 output elements across traces: exact."""
    torch = gpu_or_skip()
    from oracle import resample as ors
    from paper_2502_12350_amd import resample
    d = np.random.default_rng(nrec).standard_normal((nrec, nt_in)).astype(np.float32)
    for dt_out in (0.4e-3, 1.3e-3):
        ref = ors.resample(d, 1.0e-3, nt_out, dt_out, "nearest")
        got = resample(torch.from_numpy(d).cuda(), 1.0e-3, nt_out, dt_out, "nearest")
        assert np.array_equal(got.cpu().numpy(), ref)
