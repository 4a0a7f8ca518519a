"""Small 3D grids and 2D grids. Grids whose stencil launch is split into chunks of one to seven levels (fewer work-groups
than the GPU holds at once): the gradient in full storage against the FP64 oracle, and
checkpointing and the space store with every patch exact against full storage bit for bit,
with receivers inside the volume. The (min, max) partials of split patch layers give the
encoder the metadata that the standalone normalisation computes."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import wave as ow
from paper_2304_04781_amd import _lib as L
from paper_2304_04781_amd.compressor import Autoencoder
from paper_2304_04781_amd.solver import WaveSolver

pytestmark = pytest.mark.gpu


# chunks of 1, 1, 1, 3, 5 and (2D) 1 levels; partials per patch layer of 2, 2, -, 4, - levels
@pytest.mark.parametrize("shape", [(8, 16, 16), (16, 24, 72), (21, 10, 67), (56, 128, 136), (60, 131, 70), (131, 1, 65)])
@pytest.mark.parametrize("nsrc", [1, 2])
def test_small_grids(shape, nsrc):
    print("case", shape, nsrc, flush=True)
    nz, ny, nx = shape
    nt = 24
    p = W.problem_3d(*shape, nt, f0=15.0, sponge=2, name="small") if ny > 1 else W.problem_2d_small(nt)
    rng = np.random.default_rng(3)
    p.nz, p.ny, p.nx = shape
    p.c_true = 2000.0 + 300.0 * rng.random(shape)
    p.c_start = 2000.0 + 300.0 * rng.random(shape)
    p.c_ref = float(p.c_true.max())
    p.src = np.stack([np.array([min(4, nz - 1), ny // 2, nx // 2 - s]) for s in range(nsrc)]).astype(np.int32)
    p.rec = np.stack([rng.integers(0, nz, 40), rng.integers(0, ny, 40), rng.integers(0, nx, 40)], axis=1).astype(np.int32)
    p.rec[1] = p.rec[0]
    p.wavelet = rng.standard_normal((nsrc, nt)) / p.dx ** p.dims
    p.noise = rng.standard_normal((nsrc, nt, 40))
    for name in ("c_true", "c_start", "wavelet"):
        setattr(p, name, np.asarray(getattr(p, name), np.float32).astype(np.float64))
    sol = ow.solver_for(p)
    d, sigma, _ = ow.observed_data(sol, p)
    J_o, g_o, _, _ = ow.gradient(sol, p.c_start, p.wavelet, p.src, p.rec, d, sigma, src_w=p.src_w)
    full = WaveSolver.for_problem(p)
    full.set_storage(L.STORE_FULL)
    J0, g0 = full.gradient(p.c_start, p.wavelet, d, sigma)
    assert abs(J0 - J_o) / J_o < 1e-5
    err = np.linalg.norm(g0.cpu().numpy() - g_o) / np.linalg.norm(g_o)
    assert err < 1e-4, err
    dc = p.c_start * 0.01 * rng.standard_normal(shape)
    H0, F0 = full.hessvec(p.c_start, dc), full.hessvec(p.c_start, dc, gauss_newton=False)
    ck = WaveSolver.for_problem(p)
    ck.set_storage(L.STORE_CHECKPOINT, n_checkpoints=4)
    J, g = ck.gradient(p.c_start, p.wavelet, d, sigma)
    assert J == J0 and torch.equal(g, g0)
    assert torch.equal(ck.hessvec(p.c_start, dc), H0)
    if ny > 1 and nz % 8 == 0 and ny % 8 == 0 and nx % 8 == 0:
        net = Autoencoder(W.ae_init(2048, 512, 32, seed=4))
        ae = WaveSolver.for_problem(p)
        L.wv_set_ae_exceptions(ae.ctx, nz * ny * nx // 512)
        ae.set_storage(L.STORE_AE_BF16, ae=net)
        J, g = ae.gradient(p.c_start, p.wavelet, d, sigma)
        assert J == J0 and torch.equal(g, g0)
        assert torch.equal(ae.hessvec(p.c_start, dc), H0)
        assert torch.equal(ae.hessvec(p.c_start, dc, gauss_newton=False), F0)
        # latents only: the stored e is the codec's round trip, whose metadata is exact
        L.wv_set_ae_exceptions(ae.ctx, 0)
        ae.set_storage(L.STORE_AE_BF16, ae=net)
        _, last, cap = ae.forward(p.c_start, p.wavelet, final_state=True, capture_every=1)
        P = nz * ny * nx // 512
        z = torch.empty((P, 32), dtype=torch.int16, device="cuda")
        m = torch.empty((P, 4, 2), dtype=torch.float32, device="cuda")
        out = torch.zeros((4,) + shape, dtype=torch.float32, device="cuda")
        for n in (1, nt - 1):
            got = ae.load_e(n)
            for s in range(nsrc):
                L.ae_encode(net.handle, ae.grid, cap[n - 1, s].contiguous(), L.LATENT_BF16, z, m)
                L.ae_decode(net.handle, ae.grid, z, m, None, L.LATENT_BF16, 1, out)
                assert torch.equal(got[s], out[0]), (n, s)
        ae.close()
    ck.close()
    full.close()


# 2D grids step up to 8 levels per launch in 8 x 16 cell cores: sizes below, at and past a core
# and past the largest grid stepped so, horizons around a launch, captures that cut launches
@pytest.mark.parametrize("shape,nt", [((8, 16), 2), ((7, 15), 9), ((9, 17), 8), ((40, 130), 26), ((33, 70), 17),
                                      ((730, 730), 10)])
@pytest.mark.parametrize("nsrc", [1, 2])
def test_2d_grids(shape, nt, nsrc):
    print("case", shape, nt, nsrc, flush=True)
    nz, nx = shape
    rng = np.random.default_rng(4)
    p = W.problem_2d_small(nt)
    p.nz, p.ny, p.nx, p.nt, p.sponge = nz, 1, nx, nt, 2
    p.c_true = 2000.0 + 300.0 * rng.random((nz, 1, nx))
    p.c_start = 2000.0 + 300.0 * rng.random((nz, 1, nx))
    p.c_ref = float(p.c_true.max())
    p.src = np.array([[min(4, nz - 1), 0, nx // 2], [0, 0, nx - 1]], dtype=np.int32)[:nsrc]
    p.rec = np.stack([rng.integers(0, nz, 60), np.zeros(60, int), rng.integers(0, nx, 60)], axis=1).astype(np.int32)
    p.rec[:6] = [[0, 0, 0], [nz - 1, 0, nx - 1], [min(7, nz - 1), 0, min(15, nx - 1)], [min(8, nz - 1), 0, min(16, nx - 1)],
                 [2, 0, nx // 2], [2, 0, nx // 2]]
    p.wavelet = rng.standard_normal((nsrc, nt)) / p.dx ** 2
    p.noise = rng.standard_normal((nsrc, nt, 60))
    for name in ("c_true", "c_start", "wavelet"):
        setattr(p, name, np.asarray(getattr(p, name), np.float32).astype(np.float64))
    sol = ow.solver_for(p)
    d, sigma, _ = ow.observed_data(sol, p)
    J_o, g_o, _, e_o = ow.gradient(sol, p.c_start, p.wavelet, p.src, p.rec, d, sigma, src_w=p.src_w)
    full = WaveSolver.for_problem(p)
    full.set_storage(L.STORE_FULL)
    J0, g0 = full.gradient(p.c_start, p.wavelet, d, sigma)
    assert abs(J0 - J_o) / J_o < 1e-5
    assert np.linalg.norm(g0.cpu().numpy() - g_o) / np.linalg.norm(g_o) < 1e-4
    dc = (p.c_start * 0.01 * rng.standard_normal((nz, 1, nx))).astype(np.float32).astype(np.float64)
    H_o = ow.hessvec_gn(sol, p.c_start, dc, e_o, p.rec, sigma)
    H0 = full.hessvec(p.c_start, dc)
    assert np.linalg.norm(H0.cpu().numpy() - H_o) / np.linalg.norm(H_o) < 1e-4
    assert torch.isfinite(full.hessvec(p.c_start, dc, gauss_newton=False)).all()
    for slots in (1, 3, 40):
        ck = WaveSolver.for_problem(p)
        ck.set_storage(L.STORE_CHECKPOINT, n_checkpoints=slots)
        J, g = ck.gradient(p.c_start, p.wavelet, d, sigma)
        assert J == J0 and torch.equal(g, g0), slots
        assert torch.equal(ck.hessvec(p.c_start, dc), H0), slots
        ck.close()
    # states captured one by one (a launch per step) against launches of several steps
    tr1, last1, cap = full.forward(p.c_start, p.wavelet, final_state=True, capture_every=1)
    tr, last, cap3 = full.forward(p.c_start, p.wavelet, final_state=True, capture_every=3)
    assert torch.equal(tr, tr1) and torch.equal(last, last1) and torch.equal(cap3, cap[2::3])
    levels = [nt, 1] if nt > 1 else [1]
    e = full.forward_e(p.c_start, p.wavelet, levels)
    assert torch.equal(e[0], last[:, 0]) and torch.equal(e[1], cap[0][:, 0])
    full.close()
