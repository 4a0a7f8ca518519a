"""The elliptic solve behind prior draws and the prior preconditioner, over the shapes where
its launches differ (four cells or one per lane, ragged tiles, one or many levels per chunk,
2D, products stored or formed twice): the residual of the returned draw in float64, the iteration limit, and repeatability.
The float32 recurrence's residual (1e-6) is off the true one by the rounding of the residual
updates, about sqrt(iterations) x 61 x 6e-8 (61: the operator's largest row sum at theta /
dx^2 = 5): 2e-5 bounds it."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2304_04781_amd import _lib as L
from paper_2304_04781_amd.solver import WaveSolver

pytestmark = pytest.mark.gpu


def operator(u, alpha, t):
    """(A u) in float64: alpha (u - sum over inner faces of t (u_nb - u))."""
    out = u.copy()
    for a in range(3):
        d = t[a] * np.diff(u, axis=a)
        lo, hi = [slice(None)] * 3, [slice(None)] * 3
        lo[a], hi[a] = slice(0, -1), slice(1, None)
        out[tuple(lo)] -= d
        out[tuple(hi)] += d
    return alpha * out


@pytest.mark.parametrize("shape", [(2, 3, 4), (5, 9, 7), (33, 17, 128), (24, 40, 132), (9, 130, 260), (70, 8, 31),
                                   (61, 1, 96), (40, 1, 33), (96, 96, 96), (190, 180, 184), (185, 184, 187)])
def test_prior_draw_residual(shape):
    print("case", shape, flush=True)
    nz, ny, nx = shape
    dx, theta, alpha = 20.0, (2000.0, 1500.0, 1000.0), 3e-4
    s = WaveSolver(nz, ny, nx, dx, 1e-3, 2, 0, 0.0, [[0, 0, 0]], [])
    rng = np.random.default_rng(1)
    c0 = np.zeros(shape, np.float32)
    s.set_prior(alpha, theta, c0)
    w = torch.tensor(rng.standard_normal(shape), dtype=torch.float32, device="cuda")
    x, it, rel = s.prior_sample(w)
    assert it > 0 and rel <= 1e-6
    vol = dx ** (3 if ny > 1 else 2)
    b = w.cpu().numpy().astype(np.float64) / np.sqrt(vol)
    r = operator(x.cpu().numpy().astype(np.float64), alpha, [t / dx ** 2 for t in theta]) - b
    assert np.linalg.norm(r) / np.linalg.norm(b) < 2e-5
    x2, it2, rel2 = s.prior_sample(w)
    assert it2 == it and rel2 == rel and torch.equal(x, x2)
    # limits below, at and above a batch of queued iterations
    for limit in (1, 7, 8, 9, 16, 17):
        xl, itl, rell = s.prior_sample(w, maxit=limit)
        assert itl == min(limit, it), limit
        assert (rell > 1e-6) == (it > limit), limit
        if it <= limit:
            assert torch.equal(xl, x), limit
    z, it0, rel0 = s.prior_sample(torch.zeros_like(w))
    assert it0 == 0 and rel0 == 0.0 and torch.count_nonzero(z) == 0
    s.close()
