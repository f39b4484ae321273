"""The row kernels over every patch side from 9 to 37 (each class of taps per lane, whole and
partial last slots), in runs of four rows and in single rows, against the FP64 oracle (eq. 6,
eq. 8), for each storage type and direction.  The tolerance is that of the parity tests."""
import sys

import numpy as np
import pytest

import wfsynth as ws
from gpu_common import TOL, rel, oracle_for, gpu_operator, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("run", [1, 4])
def test_patch_sides(store, run):
    n, rows, cell = 64, 384, np.radians(2.0) / 64
    r = np.random.default_rng(1)
    du = 299_792_458.0 / 1.28e9 / (2 * n * cell)          # metres per grid cell
    at = np.repeat(r.integers(-9, 10, (rows // run, 2)), run, 0)
    uvw = np.concatenate([(at + r.uniform(-0.05, 0.05, (rows, 2))) * du,
                          np.repeat(r.uniform(-1000, 1000, rows // run), run)[:, None]], 1)
    obs = ws.Observation("sides", uvw, np.array([1.28e9]), n, n, cell)
    orc = oracle_for(obs, 1)
    sides = {g.shape[1] for _, _, _, g in orc.patches(np.arange(rows))}
    assert sides >= set(range(9, 39, 2))
    op = gpu_operator(obs, 1, store=store)
    x = r.standard_normal((n, n)).astype(np.float32)
    v = (r.standard_normal(rows) + 1j * r.standard_normal(rows)).astype(np.complex64)
    x64, v64 = x.astype(np.float64), v.astype(np.complex128)
    for name, got, ref in (("psf", op.psf_apply(to_dev(x[None]))[0], orc.psf(x64)),
                           ("forward", op.forward(to_dev(x[None])), orc.forward(x64)),
                           ("adjoint", op.adjoint(to_dev(v))[0], orc.adjoint(v64))):
        err = rel(got.cpu().numpy(), ref)
        print(f"[gpu] {store} run {run} {name}: {err:.1e}", file=sys.stderr, flush=True)
        assert err <= TOL[store]
