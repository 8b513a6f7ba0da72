"""Kernels that must not spill vector registers (compiled for the device here, no GPU needed)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_row_reductions_of_16_bit_types_keep_their_registers(tmp_path):
    """A compiler that vectorises their loops over single elements spills 130 to 150 registers."""
    from paper_1810_08723_amd.build import COMMON
    src = tmp_path / "rows.hip"
    header = os.path.join(ROOT, "paper_1810_08723_amd", "csrc", "red_launch.hpp")
    kernels = [("DT_I16", "R_ANY"), ("DT_I16", "R_MAX"), ("DT_U16", "R_MIN"), ("DT_F16", "R_ALL")]
    src.write_text(f'#include "{header}"\nnamespace ocn {{\n' + "".join(
        f"template __global__ void red_rows_kernel<{s}, {op}>(const RedArgs);\n" for s, op in kernels) + "}\n")
    r = subprocess.run([HIPCC, *COMMON, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
                        str(src), "-o", os.devnull], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spills = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    rows = [(n, k) for n, k in zip(names, spills) if "red_rows_kernel" in n]
    assert len(rows) == len(kernels) and all(k == 0 for _, k in rows), rows
