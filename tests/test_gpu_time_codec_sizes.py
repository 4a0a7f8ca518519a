"""Windows of the time scheme large enough for the fused kernels against the same blocks a slab of z rows
at a time, which take the general products: the same latents, metadata and levels, bit for bit."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2304_04781_amd import _lib as L
from paper_2304_04781_amd.compressor import Autoencoder

pytestmark = pytest.mark.gpu


# 8568, 13125, 12800, 12480 and 16384 vectors; 128 and 64 to a work-group, blocks along x in groups of 1 to 8
@pytest.mark.parametrize("shape,nsrc", [((68, 96, 84), 1), ((100, 100, 84), 1), ((64, 64, 100), 2), ((104, 120, 64), 1),
                                        ((64, 64, 128), 2)])
@pytest.mark.parametrize("nvalid", [1, 8, 9, 31, 32])
def test_fused_time_codec(shape, nsrc, nvalid):
    print("case", shape, nsrc, nvalid, flush=True)
    nz, ny, nx = shape
    B = nz * ny * nx // 64
    g = L.make_grid(nz, ny, nx, 10.0, 1e-3, 32, 8, 3000.0, nsrc, 0)
    gen = torch.Generator(device="cuda").manual_seed(7)
    e = torch.randn((32, nsrc) + shape, generator=gen, device="cuda")
    e[:, :, : nz // 2] *= 1e-9  # ranges below the floor
    e[nvalid:] = float("nan")  # never read
    net = Autoencoder(W.ae_init(2048, 512, 32, seed=4))
    z = torch.empty((nsrc, B, 32), dtype=torch.int16, device="cuda")
    m = torch.empty((nsrc, B, 2), device="cuda")
    out = torch.full_like(e, -7.0)
    L.ae_time_encode(net.handle, g, e, nvalid, z, m)
    L.ae_time_decode(net.handle, g, z, m, nvalid, out)
    assert (out[nvalid:] == -7.0).all()
    step = 16
    g1 = L.make_grid(step, ny, nx, 10.0, 1e-3, 32, 8, 3000.0, 1, 0)
    n1 = step * ny * nx // 64
    for s in range(nsrc):
        for z0 in range(0, nz - step + 1, step):
            part = e[:, s:s + 1, z0:z0 + step].contiguous()
            z1 = torch.empty((n1, 32), dtype=torch.int16, device="cuda")
            m1 = torch.empty((n1, 2), device="cuda")
            o1 = torch.empty_like(part)
            L.ae_time_encode(net.handle, g1, part, nvalid, z1, m1)
            L.ae_time_decode(net.handle, g1, z1, m1, nvalid, o1)
            b0 = z0 // 4 * (ny // 4) * (nx // 4)
            assert torch.equal(m[s, b0:b0 + n1], m1), (s, z0)
            assert torch.equal(z[s, b0:b0 + n1], z1), (s, z0)
            assert torch.equal(out[:nvalid, s:s + 1, z0:z0 + step], o1[:nvalid]), (s, z0)
