"""The training step over layer widths and batches with remainders in every tile: the update against Adam in
float64 on the gradients that the step reports, the gradients against float32 products of the same
operands, the run of several batches against single steps, and the bf16 copies against a network made from the parameters."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2304_04781_amd import _lib as L
from paper_2304_04781_amd.compressor import Autoencoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hid,lat,B,weighting", [(64, 32, 32, 0), (576, 64, 96, 1), (512, 32, 992, 1), (128, 64, 4128, 0),
                                                 (512, 32, 4096, 1)])
def test_train_sizes(hid, lat, B, weighting):
    print("case", hid, lat, B, weighting, flush=True)
    rng = np.random.default_rng(6)
    init = W.ae_init(2048, hid, lat, seed=4)
    flat = np.concatenate([np.asarray(init[k], np.float32).ravel() for l in "1234" for k in ("W" + l, "b" + l)])
    ns = 3 * B
    y = torch.tensor(rng.random((ns, 2048), dtype=np.float32), device="cuda").to(torch.bfloat16)
    yt = y.view(torch.int16)
    meta = torch.tensor(rng.random((ns, 4, 2), dtype=np.float32) + 0.5, device="cuda")
    perm = torch.tensor(rng.permutation(ns).astype(np.int32), device="cuda")
    cfg = L.train_cfg(epochs=1, batch=B, weighting=weighting)
    net, run = Autoencoder(init, 2048, hid, lat), Autoencoder(init, 2048, hid, lat)
    for n in (net, run):
        L.ae_set_beta(n.handle, np.ones(4))
    m, v, losses = np.zeros(flat.size), np.zeros(flat.size), []
    for k in range(3):
        w0 = L.ae_get_params(net.handle).astype(np.float64)
        idx = perm[k * B:(k + 1) * B].contiguous()
        loss, g = L.ae_train_step(net.handle, yt, idx, B, cfg.lr, cfg, want_grads=True, meta=meta)
        losses.append(loss)
        if k == 0:
            _check_grads(flat, hid, lat, y[idx.long()].float(), meta[idx.long()] if weighting else None, g, loss)
        g = g.astype(np.float64)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        step = cfg.lr * (m / (1 - 0.9 ** (k + 1))) / (np.sqrt(v / (1 - 0.999 ** (k + 1))) + 1e-8)
        w1 = L.ae_get_params(net.handle)
        # the update is at most 10 lr; its float32 evaluation is good to some 1e-4 of it where 1 - b1, 1 - b2
        # and the corrections are rounded (1 - 0.999 to 5e-5 of itself), and w to half an ulp
        tol = 2e-4 * np.abs(step) + 2e-7 * np.abs(w0) + 1e-9
        assert (np.abs(w1 - (w0 - step)) <= tol).all()
    total = L.ae_train(run.handle, yt, ns, cfg, perm, meta=meta)
    assert np.array_equal(L.ae_get_params(run.handle), L.ae_get_params(net.handle))
    assert total[0] == np.float32(sum(losses) / 3)
    # both copies of the weights: one more step from the trained network and from its parameters
    # (every gradient reads W or W^T of all layers)
    again = Autoencoder(init, 2048, hid, lat)
    L.ae_set_beta(again.handle, np.ones(4))
    L.ae_set_params(again.handle, L.ae_get_params(run.handle))
    a = L.ae_train_step(run.handle, yt, perm[:B].contiguous(), B, 0.0, cfg, want_grads=True, meta=meta)
    b = L.ae_train_step(again.handle, yt, perm[:B].contiguous(), B, 0.0, cfg, want_grads=True, meta=meta)
    assert a[0] == b[0] and np.array_equal(a[1], b[1])


def _check_grads(flat, hid, lat, y, meta, g, loss):
    """Gradients of the loss by autograd in float32 on bf16-rounded weights; the step rounds its activations
    and deltas to bf16 (2^-9 relative each, some ten roundings along the chain): 2 percent of each layer's norm."""
    dims, o, p = [2048, hid, lat, hid, 2048], 0, []
    for fi, fo in zip(dims[:-1], dims[1:]):
        w = torch.tensor(flat[o:o + fi * fo].reshape(fi, fo), device="cuda").to(torch.bfloat16).float()
        b = torch.tensor(flat[o + fi * fo:o + fi * fo + fo], device="cuda")
        p += [w.requires_grad_(), b.requires_grad_()]
        o += fi * fo + fo
    h = torch.nn.functional.gelu(y @ p[0] + p[1])
    h = torch.nn.functional.gelu((h @ p[2] + p[3]) @ p[4] + p[5])
    d = (h @ p[6] + p[7] - y).view(-1, 4, 512)
    w = meta[:, :, 1] ** 2 if meta is not None else torch.ones(d.shape[:2], device="cuda")
    ref = ((d * d).mean(2) * w).sum() / w.sum()
    ref.backward()
    assert abs(loss - ref.item()) < 0.01 * ref.item()
    o = 0
    for q in p:
        part = torch.tensor(g[o:o + q.numel()], device="cuda").view(q.shape)
        assert torch.norm(part - q.grad) < 0.02 * torch.norm(q.grad), q.shape
        o += q.numel()
