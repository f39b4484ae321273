"""Work items cut into pieces for the row kernels' launches: rows crowded into one grid cell
or one tile, at counts around a piece's smallest size and an item's largest, against the FP64
oracle (eq. 6, eq. 8), for stored G and G on the fly."""
import sys

import numpy as np
import pytest

import wfsynth as ws
from gpu_common import TOL, rel, oracle_for, gpu_operator, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 63, 65, 1025, 5000])
@pytest.mark.parametrize("spread,strategy", [(0.1, "G"), (12.0, "G"), (12.0, "otf")])
def test_crowded_rows(rows, spread, strategy):
    n, cell = 64, np.radians(2.0) / 64
    r = np.random.default_rng(rows)
    du = 299_792_458.0 / 1.28e9 / (2 * n * cell)          # metres per grid cell
    uvw = np.stack([r.uniform(-spread, spread, rows) * du, r.uniform(-spread, spread, rows) * du,
                    r.uniform(-600, 600, rows)], 1)
    obs = ws.Observation("crowded", uvw, np.array([1.28e9]), n, n, cell)
    print(f"[gpu] {rows} rows within {spread} cells, {strategy}", file=sys.stderr, flush=True)
    op, orc = gpu_operator(obs, 1, strategy=strategy), oracle_for(obs, 1)
    x = r.standard_normal((n, n)).astype(np.float32)
    v = (r.standard_normal(rows) + 1j * r.standard_normal(rows)).astype(np.complex64)
    x64, v64 = x.astype(np.float64), v.astype(np.complex128)
    assert rel(op.psf_apply(to_dev(x[None])).cpu().numpy()[0], orc.psf(x64)) <= TOL["f32"]
    assert rel(op.forward(to_dev(x[None])).cpu().numpy(), orc.forward(x64)) <= TOL["f32"]
    assert rel(op.adjoint(to_dev(v)).cpu().numpy()[0], orc.adjoint(v64)) <= TOL["f32"]
