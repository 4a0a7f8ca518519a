"""The codec kernels chosen by the number of patches (16, 32, 64 or 128 per work-group, the
hidden layer split or whole) against each other: patches are independent, so a state coded
whole must give, bit for bit, what its layers of patches give when coded one by one. The
exception patches of small and larger grids against a direct selection from the ranges."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2304_04781_amd import _lib as L
from paper_2304_04781_amd.compressor import Autoencoder
from paper_2304_04781_amd.solver import WaveSolver

pytestmark = pytest.mark.gpu


def grid_of(shape, nsrc=1):
    return L.make_grid(*shape, 20.0, 1e-3, 10, 0, 1.0, nsrc, 0)


def state_of(shape, seed):
    """Smooth fields whose scale spreads over six decades from patch to patch."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((4,) + shape, generator=gen, device="cuda")
    for d in (1, 2, 3):
        x = x + x.roll(1, d) + x.roll(2, d)
    env = torch.exp(-14.0 * torch.rand([n // 8 for n in shape], generator=gen, device="cuda"))
    for d in range(3):
        env = env.repeat_interleave(8, dim=d)
    return (x * env).contiguous()


def encode(net, shape, x, fmt):
    P = shape[0] * shape[1] * shape[2] // 512
    z = torch.full((P, 32), 0x55, dtype=torch.uint8 if fmt else torch.int16, device="cuda")
    m = torch.full((P, 4, 2), float("nan"), device="cuda")
    q = torch.full((P,), float("nan"), device="cuda") if fmt else None
    L.ae_encode(net.handle, grid_of(shape), x, fmt, z, m, q)
    return z, m, q


# whole: 2040 and 2054, 4080 and 4104, 8160 and 8208, 16320 and 16416 patches
@pytest.mark.parametrize("shape", [(80, 96, 136), (104, 632, 16), (160, 96, 136), (144, 152, 96), (160, 136, 192),
                                   (144, 152, 192), (320, 136, 192), (288, 152, 192)])
@pytest.mark.parametrize("fmt", [L.LATENT_BF16, L.LATENT_FP8])
def test_whole_state_equals_its_layers(shape, fmt):
    print("case", shape, fmt, flush=True)
    net = Autoencoder(W.ae_init(2048, 512, 32, seed=4), beta=[1e-5] * 4)
    x = state_of(shape, 3)
    z, m, q = encode(net, shape, x, fmt)
    out = torch.full_like(x, float("nan"))
    L.ae_decode(net.handle, grid_of(shape), z, m, q, fmt, 15, out)
    assert torch.isfinite(out).all()
    one = (8,) + shape[1:]
    n = one[1] * one[2] // 64
    for k in range(0, shape[0] // 8, 3):
        part = x[:, 8 * k:8 * k + 8].contiguous()
        zk, mk, qk = encode(net, one, part, fmt)
        s = slice(k * n, (k + 1) * n)
        assert torch.equal(z[s], zk) and torch.equal(m[s], mk), k
        assert q is None or torch.equal(q[s], qk), k
        ok = torch.zeros_like(part)
        L.ae_decode(net.handle, grid_of(one), zk, mk, qk, fmt, 15, ok)
        assert torch.equal(out[:, 8 * k:8 * k + 8], ok), k


def test_encode_under_graph_capture():
    """A captured encode of few patches replays on new contents of its input."""
    shape = (24, 40, 56)
    net = Autoencoder(W.ae_init(2048, 512, 32, seed=4), beta=[1e-5] * 4)
    x = state_of(shape, 1)
    z = torch.zeros((210 // 2, 32), dtype=torch.int16, device="cuda")
    m = torch.zeros((210 // 2, 4, 2), device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.ae_encode(net.handle, grid_of(shape), x, L.LATENT_BF16, z, m)
    for seed in (2, 3, 4):
        x.copy_(state_of(shape, seed))
        g.replay()
        torch.cuda.synchronize()
        ze, me, _ = encode(net, shape, x, L.LATENT_BF16)
        assert torch.equal(z, ze) and torch.equal(m, me), seed


@pytest.mark.parametrize("shape,K", [((16, 24, 40), 1), ((40, 48, 56), 7), ((64, 64, 128), 64), ((64, 64, 136), 65),
                                     ((96, 96, 96), 100)])
@pytest.mark.parametrize("nsrc", [1, 2])
def test_exception_patches(shape, K, nsrc):
    """The stored e is exact on the K patches of the largest ranges (compared by the top 14
    bits, lower patches first) and the decoded one elsewhere."""
    print("case", shape, K, nsrc, flush=True)
    nz, ny, nx = shape
    p = W.problem_3d(*shape, 12, f0=15.0, sponge=2, name="exc")
    rng = np.random.default_rng(5)
    p.src = np.array([[4, ny // 2, nx // 2], [6, ny // 3, nx // 3]], dtype=np.int32)[:nsrc]
    p.wavelet = rng.standard_normal((nsrc, 12)) / p.dx ** 3
    net = Autoencoder(W.ae_init(2048, 512, 32, seed=4), beta=[1e-12] * 4)
    s = WaveSolver.for_problem(p)
    L.wv_set_ae_exceptions(s.ctx, K)
    s.set_storage(L.STORE_AE_BF16, ae=net)
    _, _, cap = s.forward(p.c_start, p.wavelet, capture_every=1)
    for n in (2, 11):
        got = s.load_e(n)
        for q in range(nsrc):
            x = cap[n - 1, q].contiguous()
            z, m, _ = encode(net, shape, x, L.LATENT_BF16)
            want = torch.zeros_like(x)
            L.ae_decode(net.handle, grid_of(shape), z, m, None, L.LATENT_BF16, 1, want)
            key = m[:, 0, 1].contiguous().view(torch.int32) >> 18
            pick = torch.sort(key, descending=True, stable=True)[1][:K].cpu().numpy()
            e = want[0].clone()
            for i in pick:
                pz, py, px = i // (ny // 8 * (nx // 8)), i // (nx // 8) % (ny // 8), i % (nx // 8)
                b = (slice(8 * pz, 8 * pz + 8), slice(8 * py, 8 * py + 8), slice(8 * px, 8 * px + 8))
                e[b] = x[0][b]
            assert torch.equal(got[q], e), (n, q)
    s.close()
