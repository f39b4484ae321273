"""Every line length of the row and column passes below the long ones (16 to 1024 points),
with rows and columns of different lengths and pruning tiles smaller and larger than a
pass's step, against the FP64 oracle: F Z_p x element-wise (unmasked passes), Phi x,
Phi^dag y and Phi^dag Phi x twice in a row (masked passes; the grid is left cleared)."""
import sys

import numpy as np
import pytest

import wfsynth as ws
from gpu_common import TOL, rel, oracle_for, gpu_operator, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,tile", [(8, 16, 8), (16, 8, 32), (32, 64, 8), (64, 32, 64),
                                        (128, 256, 8), (256, 128, 64), (512, 128, 16),
                                        (64, 512, 32), (512, 1024, 8)])
def test_line_lengths(nx, ny, tile):
    obs = ws.widefield(n=max(nx, ny), nvis=3000, fov_deg=2.0, sky=False)
    obs.nx, obs.ny = nx, ny
    print(f"[gpu] {nx} x {ny}, tile {tile}", file=sys.stderr, flush=True)
    op = gpu_operator(obs, 2, tile=tile, smax=15)
    orc = oracle_for(obs, 2, smax=15)
    r = np.random.default_rng(nx + ny)
    x = r.standard_normal((ny, nx)).astype(np.float32)
    v = (r.standard_normal(orc.M) + 1j * r.standard_normal(orc.M)).astype(np.complex64)
    xd, vd = to_dev(x[None]), to_dev(v)
    g = op.layer_grid(0, 1, xd).cpu().numpy()
    assert rel(g, orc.fwd_fft(orc.zp(1) * x.astype(np.float64))) <= 2e-6
    psf, adj = orc.psf(x.astype(np.float64)), orc.adjoint(v.astype(np.complex128))
    for _ in range(2):
        assert rel(op.psf_apply(xd).cpu().numpy()[0], psf) <= TOL["f32"]
        assert rel(op.adjoint(vd).cpu().numpy()[0], adj) <= TOL["f32"]
    assert rel(op.psf_apply_re(xd).cpu().numpy()[0], psf.real) <= TOL["f32"]
    assert rel(op.forward(xd).cpu().numpy(), orc.forward(x.astype(np.float64))) <= TOL["f32"]
