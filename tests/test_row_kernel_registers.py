"""Registers of the row kernels as compiled for gfx950 (no GPU needed): none uses scratch memory,
and those of the layer-batched sweep let a compute unit hold at least the workgroups that their
forms are chosen for.  A workgroup is eight wavefronts, two on each SIMD of 512 registers."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MK = (2, 4, 7, 12, 16, 22)                      # taps per lane of the patch classes
# workgroups per compute unit: [FP32, FP16, BF16][fused, de-gridding, gridding][class]
LEAST = [[(4, 2, 2, 2, 2, 1), (4, 3, 2, 2, 2, 1), (4, 3, 2, 2, 2, 2)],
         [(4, 3, 2, 2, 2, 2), (4, 4, 3, 2, 2, 2), (4, 4, 3, 2, 2, 2)],
         [(4, 3, 2, 2, 2, 1), (4, 4, 3, 2, 2, 1), (4, 4, 3, 3, 2, 2)]]


def _registers():
    """{kernel: (VGPRs, bytes of scratch)} of k_grid.hip's device code."""
    spec = importlib.util.spec_from_file_location(
        "wf_build_lib", os.path.join(ROOT, "paper_2605_26347_amd", "build_lib.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    try:
        hipcc = b._hipcc()
    except RuntimeError as e:
        pytest.skip(str(e))
    r = subprocess.run([hipcc] + b._common() + b.SOURCES["k_grid.hip"] + [
        "--cuda-device-only", "-S", os.path.join(b.CSRC, "k_grid.hip"), "-o", "-"],
        capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = {}
    for entry in r.stdout.split("amdhsa.kernels:")[1].split("  - .agpr_count")[1:]:
        get = lambda k: re.search(rf"\.{k}:\s+(\S+)", entry).group(1)  # noqa: E731
        out[get("name")] = (int(get("vgpr_count")), int(get("private_segment_fixed_size")))
    return out


@pytest.mark.timeout(600)
def test_row_kernel_registers():
    regs = _registers()
    rows = {n: v for n, v in regs.items() if "k_rows" in n}
    assert len(rows) > 54
    for name, (_, scratch) in rows.items():
        assert scratch == 0, name
    for store in range(3):
        for mode in range(3):
            for mk, least in zip(MK, LEAST[store][mode]):
                (v,) = [v for n, (v, _) in rows.items()
                        if f"k_rows_sweepILi{store}ELi{mk}ELi{mode}E" in n]
                held = min(4, 512 // (-(-v // 8) * 8) // 2)
                assert held >= least, (store, mode, mk, v)
