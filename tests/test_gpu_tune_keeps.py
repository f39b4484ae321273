"""The autotuner leaves a channel's split of 1024 rows per item as it is where no other split has
other items (every item shorter than 256 rows, one item tile), for stored G and on the fly, and
still replaces one that is not among those it tries."""
import numpy as np
import pytest

import wfsynth as ws
from gpu_common import gpu_operator, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strategy", ["G", "otf"])
@pytest.mark.parametrize("rows_per_item", [1024, 200])
def test_split_without_gain_stays(strategy, rows_per_item):
    obs = ws.widefield(n=256, nvis=3000, fov_deg=2.0, sky=False)
    op = gpu_operator(obs, 2, strategy=strategy, tile=64, max_rows_per_item=rows_per_item)
    x = to_dev(np.random.default_rng(3).standard_normal((1, 256, 256)).astype(np.float32))
    ref, items = op.psf_apply_re(x).cpu().numpy(), op.plan()["nwork"]
    info = op.autotune(x, torch.empty_like(x), reps=2)
    p = op.plan()
    if rows_per_item == 1024 and strategy == "G":
        assert p["nwork"] == items
    if rows_per_item == 1024:
        assert info["retuned_chans"] == 0 and p["max_rows_per_item"] == 1024
    else:
        assert info["retuned_chans"] == 1 and p["max_rows_per_item"] in (256, 512, 1024)
    assert rel(op.psf_apply_re(x).cpu().numpy(), ref) <= 2e-6
