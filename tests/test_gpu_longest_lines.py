"""Rows and columns of 16384 points, the longest that the transforms take (their one plan with two
passes of radix 32, one column per workgroup and 512 threads a line), beside lines of 32, against
the FP64 oracle: F Z_p x element-wise (unmasked passes), Phi x, Phi^dag y and Phi^dag Phi x twice
in a row (masked passes; the grid is left cleared)."""
import sys

import numpy as np
import pytest

import wfsynth as ws
from gpu_common import TOL, rel, oracle_for, gpu_operator, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,fov", [(8192, 16, 2.0), (16, 8192, 2.0), (8192, 16, 12.0)])
def test_longest_lines(nx, ny, fov):
    obs = ws.widefield(n=8192, nvis=2000, fov_deg=fov, sky=False)
    obs.nx, obs.ny = nx, ny
    print(f"[gpu] {nx} x {ny}, {fov} degrees", file=sys.stderr, flush=True)
    op = gpu_operator(obs, 2, tile=32, smax=15)
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
