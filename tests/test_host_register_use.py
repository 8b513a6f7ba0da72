"""Kernels whose time hangs on how many registers they use (compiled for the device here, no GPU needed)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_08723_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")


def _usage(folder, kernels, header="red_launch.hpp"):
    """(kernel, its vector registers, those spilled) of each; kernels: declarations of template instances"""
    from paper_1810_08723_amd.build import COMMON
    src = folder / "kernels.hip"
    src.write_text(f'#include "{os.path.join(CSRC, header)}"\nnamespace ocn {{\n' + "".join(f"template __global__ void {k};\n" for k in kernels) + "}\n")
    r = subprocess.run([HIPCC, *COMMON, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
                        str(src), "-o", os.devnull], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    used = [int(n) for n in re.findall(r"\sVGPRs: (\d+)", r.stderr)]
    spilled = [int(n) for n in re.findall(r"\sVGPRs Spill: (\d+)", r.stderr)]
    assert len(names) == len(used) == len(spilled) == len(kernels)
    return list(zip(names, used, spilled))


def test_any_and_all_of_byte_columns(tmp_path):
    """Both forms in one kernel take 85 to 128 registers, and spill."""
    kinds = [(s, op) for s in ("DT_BOOL", "DT_I8", "DT_U8") for op in ("R_ANY", "R_ALL")] + [("DT_BOOL", "R_MIN"), ("DT_BOOL", "R_MAX")]
    use = _usage(tmp_path, [f"{k}<{s}, {op}>(const RedArgs)" for s, op in kinds for k in ("red_cols_kernel", "red_cols_bits_kernel")])
    assert all(used <= 72 and spilled == 0 for _, used, spilled in use), use     # (seven wavefronts of a SIMD)


def test_bytes_in_strips(tmp_path):
    """Sixteen 64-bit sums of a lane and the words that become them: four vectors of unsigned bytes ahead spill."""
    use = _usage(tmp_path, [f"red_strip_{k}_kernel<{s}, {op}>(const RedStripArgs)" for k in ("cols", "runs") for s in ("DT_BOOL", "DT_I8", "DT_U8")
                            for op in ("R_SUM", "R_PROD", "R_MAX", "R_ANY")])
    assert all(spilled == 0 for _, _, spilled in use), use


def test_rows_of_bytes_without_pieces(tmp_path):
    """What flat calls, and rows shorter than a vector of bytes, run: as many wavefronts as a SIMD has."""
    sigs = [f"Sig<{op}, {t}, {t}, {t}, 2>" for op in ("B_ADD", "B_MUL") for t in ("DT_I8", "DT_U8")] + ["Sig<B_LAND, DT_BOOL, DT_BOOL, DT_BOOL, 2>"]
    use = _usage(tmp_path, [f"ew_rows_kernel<{s}, false>(const RowsArgs)" for s in sigs], header="ew_kernels.hpp")
    assert all(used <= 64 and spilled == 0 for _, used, spilled in use), use
