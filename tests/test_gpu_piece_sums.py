"""Rows of a work item that is cut into pieces are still summed in FP64 before they reach the
FP32 grid: the adjoint of 20,000 rows crowded into 28^2 cells, all classes of patches, against
the FP64 oracle (eq. 8).  Whole items leave 1.74e-7 there (the FFT's and the values' own
rounding, and one FP32 addition per item and cell); with an FP32 addition per piece it is
2.33e-7.  The bound, 2.0e-7, lies between the two."""
import sys

import numpy as np
import pytest

import wfsynth as ws
from gpu_common import rel, oracle_for, gpu_operator, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_pieces_meet_in_fp64():
    n, rows, cell = 64, 20_000, np.radians(2.0) / 64
    du = 299_792_458.0 / 1.28e9 / (2 * n * cell)          # metres per grid cell
    err = []
    for seed in range(2):
        r = np.random.default_rng(seed)
        uvw = np.stack([r.uniform(-14, 14, rows) * du, r.uniform(-14, 14, rows) * du,
                        r.uniform(-600, 600, rows)], 1)
        obs = ws.Observation("crowded", uvw, np.array([1.28e9]), n, n, cell)
        op, orc = gpu_operator(obs, 1), oracle_for(obs, 1)
        v = (r.standard_normal(rows) + 1j * r.standard_normal(rows)).astype(np.complex64)
        ref = orc.adjoint(v.astype(np.complex128))
        err.append(rel(op.adjoint(to_dev(v)).cpu().numpy()[0], ref))
        print(f"[gpu] {rows} rows in 28^2 cells: {err[-1]:.2e}", file=sys.stderr, flush=True)
    assert np.sqrt(np.mean(np.square(err))) <= 2.0e-7
