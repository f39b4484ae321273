"""The holographic apply gives the same bits every time, however a tile's stencil is shared out:
few tiles (bands of them, in shares of one wavefront), several hundred (two to four shares in one
workgroup) and more than 2048 (whole stencils); and the shares' sum against the fused form (order
of FP32 additions only: 2e-6)."""
import sys

import numpy as np
import pytest

import wfsynth as ws
from gpu_common import rel, gpu_operator, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows,smax,bins", [(32, 40, 31, 1), (64, 300, 9, 2), (128, 700, 9, 1),
                                              (512, 9000, 5, 1), (512, 9000, 15, 2),
                                              (1024, 9000, 3, 1)])
def test_same_bits(n, rows, smax, bins):
    r = np.random.default_rng(n)
    cell = np.radians(1.0) / n
    half = 0.45 * 299_792_458.0 / 1.28e9 / cell          # metres at 0.9 of the grid's edge
    uvw = np.stack([r.uniform(-half, half, rows), r.uniform(-half, half, rows),
                    r.uniform(-400, 400, rows)], 1)
    obs = ws.Observation("scattered", uvw, np.array([1.28e9]), n, n, cell)
    h = gpu_operator(obs, bins, smax=smax, strategy="H")
    x = to_dev(r.standard_normal((1, n, n)).astype(np.float32))
    first = h.psf_apply(x).clone()
    print(f"[gpu] {n}^2 / {rows} rows, {bins} bins", file=sys.stderr, flush=True)
    for _ in range(20):
        assert torch.equal(h.psf_apply(x), first)
    g = gpu_operator(obs, bins, smax=smax)
    assert rel(first.cpu().numpy(), g.psf_apply(x).cpu().numpy()) <= 2e-6
