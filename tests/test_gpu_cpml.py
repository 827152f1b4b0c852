"""CPML absorbing layer on the GPU (§2.1, reading R26) against the oracle
(oracle/cpml.py): seismograms and final states with constant and variable
density, with a free surface, receivers in the band the layer reaches, the
gradient through full storage, its central-difference check, and the
layer's absorption against the sponge's."""

import numpy as np
import pytest

import oracle
import seisgen
from gpu_util import gpu_or_skip, oracle_grid, rel_l2, say
from oracle import cpml as ocpml

pytestmark = pytest.mark.gpu

SEIS_TOL = 1e-4
GRAD_TOL = 1e-3
VMAX = 4600.0   # velocity of the layer's d0, fixed (above every model's maximum)
FPEAK = 15.0


def _workload(vd, fs=False, nt=200):
    w = seisgen.workload("c4_fd_vd" if vd else "c4_fd")
    w.nt = nt
    w.wavelet = w.wavelet[:nt].copy()
    # receivers on the model faces and edges (inside the layer's reach) and inside
    rec = [[0, 0, 0], [31, 31, 31], [0, 16, 5], [16, 31, 20], [3, 4, 31], [16, 16, 10]]
    w.receivers = w.nodes_to_metres(rec + [[2 + 4 * i, 2 + 4 * j, 4] for i in range(8)
                                           for j in range(8)])
    g = oracle_grid(w)
    g.free_surface = fs
    return w, g


def _prop(w, fs, vel=None):
    torch = gpu_or_skip()
    from paper_2502_12350_amd import GridSpec, Propagator
    P = Propagator(0)
    gs = GridSpec(**w.grid_kwargs(), free_surface=fs, cpml=True, fpeak=FPEAK, cpml_vmax=VMAX)
    v = w.vel if vel is None else vel
    P.set_model(gs, torch.from_numpy(np.ascontiguousarray(v)).cuda(),
                None if w.rho is None else torch.from_numpy(w.rho).cuda())
    return P


@pytest.mark.parametrize("vd,fs", [(False, False), (True, False), (True, True)])
def test_cpml_forward_matches_oracle(vd, fs):
    torch = gpu_or_skip()
    w, g = _workload(vd, fs)
    say(f"[cpml forward] vd {vd} free surface {fs} padded {w.padded_shape} nt {w.nt}")
    ref = ocpml.forward(g, w.vel, w.rho, w.wavelet, w.sources[0], w.receivers, vmax=VMAX,
                        fpeak=FPEAK)
    P = _prop(w, fs)
    seis, fin = P.forward(torch.from_numpy(w.wavelet).cuda(), w.sources[0], w.receivers,
                          final=True)
    torch.cuda.synchronize()
    es = rel_l2(seis.cpu().numpy(), ref.seis)
    ef = rel_l2(fin[0].cpu().numpy(), ref.last)
    say(f"  seismograms rel-L2 {es:.2e}, final state {ef:.2e}")
    assert es <= SEIS_TOL and ef <= SEIS_TOL
    # the per-receiver check covers the receivers within reach of the layer
    for r in range(6):
        assert rel_l2(seis[r].cpu().numpy(), ref.seis[r]) <= 10 * SEIS_TOL


@pytest.mark.parametrize("vd,fs", [(False, False), (True, True)])
def test_cpml_gradient_matches_oracle(vd, fs):
    torch = gpu_or_skip()
    w, g = _workload(vd, fs, nt=150)
    say(f"[cpml gradient] vd {vd} free surface {fs}")
    true = (w.vel + 5.0 * w.extra["dv"]).astype(np.float32)
    dobs = ocpml.forward(g, true, w.rho, w.wavelet, w.sources[0], w.receivers, vmax=VMAX,
                         fpeak=FPEAK).seis.astype(np.float32)
    ref = ocpml.gradient(g, w.vel, w.rho, w.wavelet, w.sources[0], w.receivers, dobs,
                         vmax=VMAX, fpeak=FPEAK, illumination=True)
    P = _prop(w, fs)
    il = torch.zeros((w.nz, w.ny, w.nx), dtype=torch.float32, device="cuda")
    J, gr, seis = P.gradient(torch.from_numpy(w.wavelet).cuda(), w.sources[0], w.receivers,
                             torch.from_numpy(dobs).cuda(), ckpt="full", illum=il, seis=True)
    torch.cuda.synchronize()
    eJ = abs(float(J.item()) - ref.misfit) / ref.misfit
    eg = rel_l2(gr.cpu().numpy(), ref.grad)
    say(f"  misfit rel {eJ:.2e}, gradient rel-L2 {eg:.2e}")
    assert rel_l2(seis.cpu().numpy(), ref.seis) <= SEIS_TOL
    assert eJ <= SEIS_TOL and eg <= GRAD_TOL
    assert rel_l2(il.cpu().numpy(), ref.illum) <= SEIS_TOL


def test_cpml_gradient_finite_difference_on_gpu():
    torch = gpu_or_skip()
    w, g = _workload(True, False, nt=200)
    true = (w.vel + 5.0 * w.extra["dv"]).astype(np.float32)
    Pt = _prop(w, False, vel=true)
    wav = torch.from_numpy(w.wavelet).cuda()
    dobs = Pt.forward(wav, w.sources[0], w.receivers).clone()
    P = _prop(w, False)
    J, gr = P.gradient(wav, w.sources[0], w.receivers, dobs, ckpt="full")
    dv = w.extra["dv"].astype(np.float64)
    an = float(np.sum(gr.cpu().numpy().astype(np.float64) * dv))
    eps = 1.0

    def Jv(v):
        Q = _prop(w, False, vel=v.astype(np.float32))
        return float(Q.forward_misfit(wav, w.sources[0], w.receivers, dobs).item())

    fd = (Jv(w.vel + eps * dv) - Jv(w.vel - eps * dv)) / (2 * eps)
    say(f"[cpml FD] analytic {an:.6e} finite difference {fd:.6e}")
    assert abs(fd - an) <= 1e-3 * abs(an)


def test_cpml_absorbs_better_than_the_sponge_on_gpu():
    torch = gpu_or_skip()
    from paper_2502_12350_amd import GridSpec, Propagator
    n, N, h, c = 48, 12, 10.0, 2000.0
    dt = 0.35 * h / c
    nt = 260
    t = np.arange(nt) * dt
    arg = (np.pi * 25.0 * (t - 1.2 / 25.0)) ** 2
    wav = torch.tensor(((1 - 2 * arg) * np.exp(-arg)).astype(np.float32), device="cuda")
    src = [24 * h, 24 * h, 24 * h]
    vel = torch.full((n, n, n), c, device="cuda")
    late = {}
    for cp in (False, True):
        P = Propagator(0)
        P.set_model(GridSpec(n, n, n, h, h, h, border=N, dt=dt, nt=nt, cpml=cp, fpeak=25.0), vel)
        _, fin = P.forward(wav, src, [src], final=True)
        torch.cuda.synchronize()
        core = (slice(N, N + n),) * 3
        d = (fin[0] - fin[1]).cpu().numpy()[core]
        late[cp] = float(np.sum(d.astype(np.float64) ** 2))
    say(f"[cpml absorption] late energy cpml {late[True]:.3e} sponge {late[False]:.3e}")
    assert late[True] < 0.05 * late[False]


def test_cpml_errors():
    torch = gpu_or_skip()
    from paper_2502_12350_amd import WfdError, GridSpec, Propagator, ShotBatch
    w, g = _workload(False, False, nt=20)
    P = _prop(w, False)
    wav = torch.from_numpy(w.wavelet).cuda()
    dobs = torch.zeros((len(w.receivers), w.nt), device="cuda")
    with pytest.raises(WfdError, match="device storage"):
        P.gradient(wav, w.sources[0], w.receivers, dobs, ckpt="host")
    with pytest.raises(WfdError, match="sponge boundaries only"):
        ShotBatch([P], wav, [w.sources[0]], [w.receivers])
    Q = Propagator(0)
    with pytest.raises(WfdError, match="fpeak"):
        Q.set_model(GridSpec(**w.grid_kwargs(), cpml=True, fpeak=-1.0),
                    torch.from_numpy(w.vel).cuda())


def test_cpml_forward_ragged_multi_tile_matches_oracle():
    # 50 x 37 x 70 model with a 14-cell layer (78 x 65 x 98 padded): two x tiles
    # with a ragged tail, 18-plane z slabs marched in two chunks with queues,
    # side boxes in many 8-plane chunks; variable density
    torch = gpu_or_skip()
    from paper_2502_12350_amd import GridSpec, Propagator
    rng = np.random.default_rng(31)
    nx, ny, nz, N, nt = 50, 37, 70, 14, 100
    vel = seisgen.layered_model(31, (nx, ny, nz), 0.05)
    rho = seisgen.gardner_density(vel)
    h = 10.0
    dt = 0.4 * h / float(vel.max())
    t = np.arange(nt) * dt
    a = (np.pi * 15.0 * (t - 1.0 / 15.0)) ** 2
    wav = ((1 - 2 * a) * np.exp(-a)).astype(np.float32)
    src = [25 * h, 18 * h, 6 * h]
    rec = np.array([[h * i, h * j, h * k] for i, j, k in
                    [(0, 0, 0), (49, 36, 69), (2, 18, 3), (47, 1, 66), (25, 0, 35), (25, 36, 35)]] +
                   [[h * rng.integers(0, nx), h * rng.integers(0, ny), h * rng.integers(0, nz)]
                    for _ in range(40)])
    g = oracle.Grid(nx, ny, nz, h, h, h, border=N, dt=dt, nt=nt)
    say(f"[cpml forward ragged] padded {g.padded_shape} nt {nt}")
    ref = ocpml.forward(g, vel, rho, wav, src, rec, vmax=VMAX, fpeak=FPEAK)
    P = Propagator(0)
    P.set_model(GridSpec(nx, ny, nz, h, h, h, border=N, dt=dt, nt=nt, cpml=True, fpeak=FPEAK,
                         cpml_vmax=VMAX), torch.from_numpy(vel).cuda(), torch.from_numpy(rho).cuda())
    seis, fin = P.forward(torch.from_numpy(wav).cuda(), src, rec, final=True)
    torch.cuda.synchronize()
    es = rel_l2(seis.cpu().numpy(), ref.seis)
    ef = rel_l2(fin[0].cpu().numpy(), ref.last)
    say(f"  seismograms rel-L2 {es:.2e}, final state {ef:.2e}")
    assert es <= SEIS_TOL and ef <= SEIS_TOL


@pytest.mark.parametrize("nsnap,fs", [(1, False), (3, True), (17, False)])
def test_cpml_checkpointed_gradient_equals_full_storage_bitwise(nsnap, fs):
    # checkpoints carry the six memory variables; the layer's correction of a
    # visited step comes from the latest forward step or is recomputed from the
    # visited state, so every bit matches full storage
    torch = gpu_or_skip()
    w, g = _workload(True, fs, nt=150)
    say(f"[cpml revolve] snapshots {nsnap} free surface {fs}")
    true = (w.vel + 5.0 * w.extra["dv"]).astype(np.float32)
    wav = torch.from_numpy(w.wavelet).cuda()
    dobs = _prop(w, fs, vel=true).forward(wav, w.sources[0], w.receivers).clone()
    out = {}
    for ck in ("full", ("revolve", nsnap)):
        P = _prop(w, fs)
        il = torch.zeros((w.nz, w.ny, w.nx), dtype=torch.float32, device="cuda")
        J, gr, seis = P.gradient(wav, w.sources[0], w.receivers, dobs, ckpt=ck, illum=il, seis=True)
        torch.cuda.synchronize()
        out[str(ck)] = (float(J.item()), gr.clone(), seis.clone(), il.clone())
    (Jf, gf, sf, ilf), (Jr, gr_, sr, ilr) = out["full"], out[str(("revolve", nsnap))]
    assert Jf == Jr and Jf > 0
    assert torch.equal(sf, sr)
    assert torch.equal(gf, gr_)
    assert torch.equal(ilf, ilr)


@pytest.mark.parametrize("n,N,fs", [
    ((70, 18, 40), 8, False),    # 12-cell segments: 3 cells per thread, ragged second x tile
    ((20, 33, 18), 16, False),   # 20 cells: 5 per thread
    ((33, 20, 17), 20, True),    # 24 cells: 6 per thread, no layer above the surface
    ((24, 17, 19), 32, False),   # 36 cells: 8 groups of 5
    ((17, 18, 20), 43, False),   # 47 cells: 8 groups of 6, side rows of 94 elements
    ((18, 17, 17), 50, False),   # 54 cells: 16 groups of 6
    ((16, 12, 14), 45, False),   # slabs meet on every axis (whole axes of 102-106 cells)
    ((16, 12, 14), 45, True),    # the same with the free surface's image cells
    ((40, 30, 3), 8, True),      # a thin model: whole z axis within the layer's reach
    ((5, 40, 30), 8, False),     # thin in x: every point within reach of an x layer
])
def test_cpml_tile_shapes_match_oracle(n, N, fs):
    # every tile shape of the layer kernels, forward and adjoint; the source is
    # next to a corner of the model so that the wave is in the layers within
    # the 36 steps.  Tolerances are those of the cases above.
    torch = gpu_or_skip()
    from paper_2502_12350_amd import GridSpec, Propagator
    nx, ny, nz = n
    nt, h = 36, 10.0
    vel = seisgen.layered_model(7, n, 0.05)
    rho = seisgen.gardner_density(vel)
    dt = 0.4 * h / float(vel.max())
    t = np.arange(nt) * dt
    a = (np.pi * 40.0 * (t - 0.02)) ** 2
    wav = ((1 - 2 * a) * np.exp(-a)).astype(np.float32)
    src = [2 * h, 3 * h, min(3, nz - 1) * h]
    rec = np.array([[h * i, h * j, h * k] for i in (0, nx // 2, nx - 1)
                    for j in (0, ny - 1) for k in (1, nz - 1)])
    g = oracle.Grid(nx, ny, nz, h, h, h, border=N, dt=dt, nt=nt)
    g.free_surface = fs
    say(f"[cpml tiles] model {n} border {N} free surface {fs}")
    dobs = (0.5 * ocpml.forward(g, vel, rho, wav, src, rec, vmax=VMAX, fpeak=FPEAK).seis)
    dobs = dobs.astype(np.float32)
    ref = ocpml.gradient(g, vel, rho, wav, src, rec, dobs, vmax=VMAX, fpeak=FPEAK)
    P = Propagator(0)
    P.set_model(GridSpec(nx, ny, nz, h, h, h, border=N, dt=dt, nt=nt, cpml=True, fpeak=FPEAK,
                         cpml_vmax=VMAX, free_surface=fs), torch.from_numpy(vel).cuda(),
                torch.from_numpy(rho).cuda())
    J, gr, seis = P.gradient(torch.from_numpy(wav).cuda(), src, rec,
                             torch.from_numpy(dobs).cuda(), ckpt="full", seis=True)
    torch.cuda.synchronize()
    es, eg = rel_l2(seis.cpu().numpy(), ref.seis), rel_l2(gr.cpu().numpy(), ref.grad)
    say(f"  seismograms rel-L2 {es:.2e}, gradient {eg:.2e}")
    assert es <= SEIS_TOL and eg <= GRAD_TOL
    assert abs(float(J.item()) - ref.misfit) <= SEIS_TOL * ref.misfit


@pytest.mark.parametrize("n,N,fs", [
    ((70, 18, 40), 8, False), ((33, 20, 17), 20, True), ((24, 40, 60), 32, False),
    ((18, 17, 17), 50, False), ((16, 12, 14), 45, True), ((40, 30, 3), 8, True),
    ((5, 40, 30), 8, False), ((30, 6, 40), 8, False), ((2, 3, 4), 30, False)])
def test_cpml_forward_equals_the_gradients_forward_sweep_bitwise(n, N, fs):
    # a forward sweep keeps no correction store and forms the terms of crossing
    # layers again; the source and the receivers are on the model's edges and
    # corners, next to the crossings
    torch = gpu_or_skip()
    from paper_2502_12350_amd import GridSpec, Propagator
    nx, ny, nz = n
    nt, h = 60, 10.0
    vel = torch.from_numpy(seisgen.layered_model(7, n, 0.05)).cuda()
    dt = 0.4 * h / float(vel.max())
    t = np.arange(nt) * dt
    a = (np.pi * 40.0 * (t - 0.02)) ** 2
    wav = torch.from_numpy(((1 - 2 * a) * np.exp(-a)).astype(np.float32)).cuda()
    src = [0.0, 0.0, min(2, nz - 1) * h]
    rec = np.array([[h * i, h * j, h * k] for i in (0, nx // 2, nx - 1)
                    for j in (0, ny // 2, ny - 1) for k in (0, nz // 2, nz - 1)])
    say(f"[cpml forward] model {n} border {N} free surface {fs}")
    P = Propagator(0)
    P.set_model(GridSpec(nx, ny, nz, h, h, h, border=N, dt=dt, nt=nt, cpml=True, fpeak=FPEAK,
                         cpml_vmax=VMAX, free_surface=fs), vel)
    dobs = torch.zeros((len(rec), nt), device="cuda")
    J, _, seis = P.gradient(wav, src, rec, dobs, ckpt="full", seis=True)
    Jf, sm = P.forward_misfit(wav, src, rec, dobs, seis=True)
    assert float(J) > 0.0
    assert torch.equal(P.forward(wav, src, rec), seis)
    assert torch.equal(sm, seis) and float(Jf) == float(J)


def test_cpml_forward_workspace_holds_no_correction():
    # two volumes, six memory variables and tables of a 150^3 grid: within the
    # library's static scratch, and with a correction of the layer's 9 MB not
    torch = gpu_or_skip()
    from paper_2502_12350_amd import GridSpec, Propagator, _lib
    from paper_2502_12350_amd.api import _dptr, _xyz
    n, nt, h = 110, 20, 10.0
    vel = torch.full((n, n, n), 2500.0, device="cuda")
    wav = torch.sin(torch.arange(nt, device="cuda") * 0.5)
    P = Propagator(0)
    P.set_model(GridSpec(n, n, n, h, h, h, border=20, dt=1e-3, nt=nt, cpml=True, fpeak=FPEAK), vel)
    src, rec = _xyz([20.0, 20.0, 20.0]), _xyz([[0.0, 0.0, 0.0], [50.0, 20.0, 40.0]])
    assert P.workspace_bytes(2) <= _lib.NOALLOC_SCRATCH_BYTES
    seis = torch.zeros((2, nt), device="cuda")
    P._sync_stream()
    _lib.check(_lib.lib().wfd_forward_noalloc(P._ctx, wav.data_ptr(), _dptr(src), 2, _dptr(rec),
                                              seis.data_ptr(), None))
    assert torch.equal(seis, P.forward(wav, src, rec)) and float(seis.abs().max()) > 0.0


@pytest.mark.parametrize("n,N,fs", [
    ((18, 20, 17), 100, False),   # 104 cells: tiles of 32 lines, 4 cells per thread
    ((18, 20, 19), 150, True),    # 154 cells: 32 lines, 6 per thread
    ((20, 18, 22), 190, False),   # 194 cells: lines marched in memory, two segments
    ((6, 20, 7), 190, True),      # whole axes marched, one with image cells
    ((70, 5, 18), 200, False)])
def test_cpml_wide_layers_match_oracle(n, N, fs, monkeypatch):
    # A layer far wider than the wave gets in nt steps (at most eight cells a step):
    # the oracle keeps its first 8 nt cells, with the full layer's profile.  vmax
    # makes those cells absorb (d dt about 0.5 in the first one), so that without
    # the layer the traces would differ by far more than the tolerance.
    torch = gpu_or_skip()
    from paper_2502_12350_amd import GridSpec, Propagator
    nx, ny, nz = n
    nt, h = 5, 10.0
    T = 8 * nt
    full = ocpml.profile

    def first_cells(m, border, *args, **kw):
        a, b = full(m, N, *args, **kw)
        assert border == T
        return a[N - T:N + m + T], b[N - T:N + m + T]

    monkeypatch.setattr(ocpml, "profile", first_cells)
    vel = seisgen.layered_model(7, n, 0.05)
    dt = 0.4 * h / float(vel.max())
    vmax = 0.5 / dt * N * N * 2 * N * h / (3.0 * np.log(1.0e3))
    wav = np.cos(0.3 * np.arange(nt)).astype(np.float32)
    src = [0.0, 0.0, min(2, nz - 1) * h]
    rec = np.array([[h * i, h * j, h * k] for i in (0, min(2, nx - 1), nx - 1)
                    for j in (0, 1) for k in (0, min(3, nz - 1))])
    g = oracle.Grid(nx, ny, nz, h, h, h, border=T, dt=dt, nt=nt)
    g.free_surface = fs
    say(f"[cpml wide] model {n} border {N} free surface {fs}")
    kw = dict(vmax=vmax, fpeak=FPEAK)
    dobs = (0.5 * ocpml.forward(g, vel, None, wav, src, rec, **kw).seis).astype(np.float32)
    ref = ocpml.gradient(g, vel, None, wav, src, rec, dobs, **kw)
    open_ = ocpml.forward(g, vel, None, wav, src, rec, vmax=0.0, fpeak=FPEAK).seis
    assert rel_l2(open_, ref.seis) > 1e-2
    P = Propagator(0)
    P.set_model(GridSpec(nx, ny, nz, h, h, h, border=N, dt=dt, nt=nt, cpml=True, fpeak=FPEAK,
                         cpml_vmax=vmax, free_surface=fs), torch.from_numpy(vel).cuda())
    J, gr, seis = P.gradient(torch.from_numpy(wav).cuda(), src, rec,
                             torch.from_numpy(dobs).cuda(), ckpt="full", seis=True)
    es, eg = rel_l2(seis.cpu().numpy(), ref.seis), rel_l2(gr.cpu().numpy(), ref.grad)
    say(f"  seismograms rel-L2 {es:.2e}, gradient {eg:.2e}")
    assert es <= SEIS_TOL and eg <= GRAD_TOL
    assert abs(float(J.item()) - ref.misfit) <= SEIS_TOL * ref.misfit
    assert torch.equal(P.forward(torch.from_numpy(wav).cuda(), src, rec), seis)
