"""Many rows of narrow patches, which the row kernels launch apart from the other classes: Phi,
Phi^dag and Phi^dag Phi for each storage type, just below and above the row counts from which they
do, against the same operator on a 2000-row subset's oracle form: y_k of the forward apply against
the FP64 oracle's rows, and the adjoint against the forward by <Phi x, y> = <x, Phi^dag y> (FP32
sums: 1e-5)."""
import sys

import numpy as np
import pytest

import wfsynth as ws
from gpu_common import TOL, rel, oracle_for, gpu_operator, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store,rows", [("f32", 299_000), ("f32", 400_001), ("bf16", 1_300_001),
                                        ("bf16", 2_100_001), ("f16", 2_100_001)])
def test_narrow_rows(store, rows):
    n, cell, sub = 128, np.radians(0.1) / 128, 2000
    r = np.random.default_rng(rows)
    du = 299_792_458.0 / 1.28e9 / (2 * n * cell)          # metres per grid cell
    uvw = np.stack([r.uniform(-60, 60, rows) * du, r.uniform(-60, 60, rows) * du,
                    r.uniform(-30, 30, rows)], 1)
    w = np.zeros(1) + uvw[:, 2].mean()
    uvw[:, 2] -= w                                        # the one w-layer at zero, as the subset's
    uvw[:sub, 2] -= uvw[:sub, 2].mean()
    obs = ws.Observation("narrow", uvw, np.array([1.28e9]), n, n, cell)
    few = ws.Observation("few", uvw[:sub], np.array([1.28e9]), n, n, cell)
    op, orc = gpu_operator(obs, 1, store=store), oracle_for(few, 1)
    assert max(op.get_row(int(k))[0] for k in r.integers(0, rows, 100)) <= 11
    x = r.standard_normal((n, n)).astype(np.float32)
    y = op.forward(to_dev(x[None]))
    e = rel(y[:sub].cpu().numpy(), orc.forward(x.astype(np.float64)))
    v = torch.view_as_complex(torch.randn(rows, 2, device="cuda"))
    a = op.adjoint(v)[0].cpu().numpy().astype(np.complex128)
    left = torch.vdot(v.to(torch.complex128), y.to(torch.complex128)).item()
    right = np.vdot(a, x.astype(np.complex128))
    scale = float(v.norm()) * float(y.norm())
    p = op.psf_apply(to_dev(x[None]))[0].cpu().numpy()
    print(f"[gpu] {store} {rows} rows: forward {e:.1e}, adjointness "
          f"{abs(left - right) / scale:.1e}", file=sys.stderr, flush=True)
    assert e <= TOL[store]
    assert abs(left - right) <= 1e-5 * scale
    assert rel(p, op.adjoint(y)[0].cpu().numpy()) <= 2e-6
