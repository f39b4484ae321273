"""Gradients of the network's large batches against FP64: the FP32 sums over the batch are cut
into chains of 256 rows at most, whatever the batch.  Bounds: with such chains the worst of the
five weight gradients is off by 2.7e-7 at 16384 rows and 2.1e-7 at 65536, and the output biases
by 1.3e-7 at 16384; with chains that grow with the batch (1024 and 4096 rows; 512 for the biases)
by 3.3e-7, 3.5e-7 and 1.9e-7.  Each bound lies between the two."""
import sys

import numpy as np
import pytest

from oracle import mlp as omlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _reference(theta, x, t):
    """Gradients (weights, biases) per layer in FP64 (oracle.mlp's loss), on the device."""
    P = torch.tensor(theta, device=x.device, dtype=torch.float64)
    x, t, B = x.double(), t.double(), x.shape[0]
    W, b, o = [], [], 0
    for i, k in zip(omlp.SIZES[:-1], omlp.SIZES[1:]):
        W.append(P[o:o + i * k].view(i, k))
        b.append(P[o + i * k:o + i * k + k])
        o += i * k + k
    H, Z = [x], []
    for l in range(len(W)):
        Z.append(H[-1] @ W[l] + b[l])
        H.append(Z[-1] * 0.5 * (1 + torch.erf(Z[-1] / 2 ** 0.5)))
    e = Z[-1][:, :450] - t
    r = e.norm(dim=1) / t.norm(dim=1).clamp_min(1e-30)
    d = torch.cat([2 * e, 2 * (Z[-1][:, 450:] - torch.log10(r.clamp_min(1e-8))[:, None])], 1) / B
    g = []
    for l in range(len(W) - 1, -1, -1):
        g.insert(0, (H[l].T @ d, d.sum(0)))
        if l:
            z = Z[l - 1]
            gelu_grad = 0.5 * (1 + torch.erf(z / 2 ** 0.5)) + z * torch.exp(-z * z / 2) / (
                2 * np.pi) ** 0.5
            n = 450 if l == len(W) - 1 else d.shape[1]     # no gradient through the error output
            d = (d[:, :n] @ W[l][:, :n].T) * gelu_grad
    return g


@pytest.mark.parametrize("B,weights,biases", [(16384, 2.95e-7, 1.6e-7), (65536, 2.7e-7, None)])
def test_large_batch_gradients(B, weights, biases):
    from paper_2605_26347_amd import Network
    net = Network(seed=1)
    net.set_params(np.asarray(omlp.init(5), dtype=np.float32))
    gen = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn(B, 5, device="cuda", generator=gen)
    t = 0.1 * torch.randn(B, 450, device="cuda", generator=gen)
    _, grad = net.loss_grad(x, t)
    grad, o = grad.double(), 0
    ew, eb = [], []
    for gw, gb in _reference(net.get_params(), x, t):
        for ref, err in ((gw.reshape(-1), ew), (gb, eb)):
            got = grad[o:o + ref.numel()]
            err.append(float((got - ref).norm() / ref.norm()))
            o += ref.numel()
    print(f"[gpu] batch {B}: weights {max(ew):.2e}, output biases {eb[-1]:.2e}",
          file=sys.stderr, flush=True)
    assert max(ew) <= weights
    assert biases is None or eb[-1] <= biases
