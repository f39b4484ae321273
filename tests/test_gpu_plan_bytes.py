"""The plan's bytes of G count the work items and their pieces (each at least one entry of 32 bytes
per item), for stored G and on the fly, also after a re-split."""
import numpy as np
import pytest

import wfsynth as ws
from gpu_common import gpu_operator

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strategy", ["G", "otf"])
def test_item_tables_are_counted(strategy):
    obs = ws.widefield(n=256, nvis=20_000, fov_deg=2.0, sky=False)
    op = gpu_operator(obs, 2, strategy=strategy)
    p = op.plan()
    rows = 12.0 * p["nrows"] + (8.0 * p["ntaps"] if strategy == "G" else p["mem_khat_bytes"])
    assert p["mem_g_bytes"] >= rows + 2 * 32 * p["nwork"]
    if strategy == "G":
        op.set_bin_tiles(np.array([64, 32]))
        q = op.plan()
        assert q["nwork"] < p["nwork"]
        assert q["mem_g_bytes"] >= rows + 2 * 32 * q["nwork"]
        assert q["mem_g_bytes"] != p["mem_g_bytes"]
