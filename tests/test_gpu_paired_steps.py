"""3D grids that are stepped twice per launch where the state between is not needed: rows of up to and past
128 and 256 cells, rows that end within a lane, tiles and chunks with remainders, odd and even horizons, against
the FP64 oracle and, bit for bit, against steps taken one by one (every state captured)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import wave as ow
from paper_2304_04781_amd import _lib as L
from paper_2304_04781_amd.compressor import Autoencoder
from paper_2304_04781_amd.solver import WaveSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,nsrc,nt", [((96, 100, 90), 1, 9), ((96, 96, 96), 1, 8), ((37, 150, 145), 1, 10),
                                           ((62, 50, 260), 1, 9), ((40, 104, 96), 2, 7), ((2, 1000, 500), 1, 6),
                                           ((128, 136, 128), 1, 6)])
def test_paired_steps(shape, nsrc, nt):
    print("case", shape, nsrc, nt, flush=True)
    nz, ny, nx = shape
    p = W.problem_3d(*shape, nt, f0=15.0, sponge=2, name="pairs")
    rng = np.random.default_rng(5)
    p.c_true = 2000.0 + 300.0 * rng.random(shape)
    p.c_start = 2000.0 + 300.0 * rng.random(shape)
    p.c_ref = float(p.c_true.max())
    p.src = np.array([[min(4, nz - 1), ny // 2, nx // 2], [nz - 1, 0, 0]], dtype=np.int32)[:nsrc]
    p.rec = np.stack([rng.integers(0, nz, 200), rng.integers(0, ny, 200), rng.integers(0, nx, 200)], axis=1).astype(np.int32)
    p.rec[0], p.rec[1], p.rec[3] = [0, 0, 0], [nz - 1, ny - 1, nx - 1], p.rec[2]
    # beside the source, so that short horizons record something
    p.rec[4:20] = p.src[0] + rng.integers(-2, 3, (16, 3)) * np.array([nz > 8, 1, 1])
    p.wavelet = rng.standard_normal((nsrc, nt)) / p.dx ** p.dims
    p.noise = rng.standard_normal((nsrc, nt, 200))
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
    tr1, last1, cap = full.forward(p.c_start, p.wavelet, final_state=True, capture_every=1)
    tr, last, cap3 = full.forward(p.c_start, p.wavelet, final_state=True, capture_every=3)
    assert torch.equal(tr, tr1) and torch.equal(last, last1) and torch.equal(cap3, cap[2::3])
    tr, last, _ = full.forward(p.c_start, p.wavelet, final_state=True)
    assert torch.equal(tr, tr1) and torch.equal(last, last1)
    for slots in (1, 2, 40):
        ck = WaveSolver.for_problem(p)
        ck.set_storage(L.STORE_CHECKPOINT, n_checkpoints=slots)
        J, g = ck.gradient(p.c_start, p.wavelet, d, sigma)
        assert J == J0 and torch.equal(g, g0), slots
        assert torch.equal(ck.hessvec(p.c_start, dc), H0), slots
        ck.close()
    if nz % 8 == 0 and ny % 8 == 0 and nx % 8 == 0:
        ae = WaveSolver.for_problem(p)
        L.wv_set_ae_exceptions(ae.ctx, nz * ny * nx // 512)
        ae.set_storage(L.STORE_AE_BF16, ae=Autoencoder(W.ae_init(2048, 512, 32, seed=4)))
        J, g = ae.gradient(p.c_start, p.wavelet, d, sigma)
        assert J == J0 and torch.equal(g, g0)
        assert torch.equal(ae.hessvec(p.c_start, dc), H0)
        assert torch.equal(ae.hessvec(p.c_start, dc, gauss_newton=False), F0)
        # latents only: the stored e is the codec's round trip of the state
        L.wv_set_ae_exceptions(ae.ctx, 0)
        net = Autoencoder(W.ae_init(2048, 512, 32, seed=4))
        P = nz * ny * nx // 512
        z, m = torch.empty((P, 32), dtype=torch.int16, device="cuda"), torch.empty((P, 4, 2), device="cuda")
        q, out = torch.empty(P, device="cuda"), torch.zeros((4,) + shape, device="cuda")
        for mode, fmt in ((L.STORE_AE_BF16, L.LATENT_BF16), (L.STORE_AE_FP8, L.LATENT_FP8)):
            ae.set_storage(mode, ae=net)
            ae.forward(p.c_start, p.wavelet)
            for n in range(1, nt):
                got = ae.load_e(n)
                for s in range(nsrc):
                    L.ae_encode(net.handle, ae.grid, cap[n - 1, s].contiguous(), fmt, z, m, q)
                    L.ae_decode(net.handle, ae.grid, z, m, q, fmt, 1, out)
                    assert torch.equal(got[s], out[0]), (mode, n, s)
        ae.close()
    full.close()
