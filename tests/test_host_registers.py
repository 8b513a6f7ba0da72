"""Kernels that must not spill registers (compiled for the device here, no GPU needed)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_08723_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _spills(source, kind):
    """(kernel, registers of the kind spilled) of every kernel that a source compiles to."""
    from paper_1810_08723_amd.build import COMMON
    r = subprocess.run([HIPCC, *COMMON, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
                        str(source), "-o", os.devnull], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    counts = [int(n) for n in re.findall(kind + r" Spill: (\d+)", r.stderr)]
    assert len(names) == len(counts)
    return list(zip(names, counts))


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_row_reductions_of_16_bit_types_keep_their_registers(tmp_path):
    """A compiler that vectorises their loops over single elements spills 130 to 150 vector registers."""
    src = tmp_path / "rows.hip"
    header = os.path.join(CSRC, "red_launch.hpp")
    kernels = [("DT_I16", "R_ANY"), ("DT_I16", "R_MAX"), ("DT_U16", "R_MIN"), ("DT_F16", "R_ALL")]
    src.write_text(f'#include "{header}"\nnamespace ocn {{\n' + "".join(
        f"template __global__ void red_rows_kernel<{s}, {op}>(const RedArgs);\n" for s, op in kernels) + "}\n")
    rows = [(n, k) for n, k in _spills(src, "VGPRs") if "red_rows_kernel" in n]
    assert len(rows) == len(kernels) and all(k == 0 for _, k in rows), rows


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_generic_dtype_kernels_keep_their_arguments_out_of_registers():
    """Arguments held in scalar registers spill there by the hundred; only the elementary functions of
    complex doubles are that large by themselves."""
    kernels = [(n, k) for n, k in _spills(os.path.join(CSRC, "ew_interp.hip"), "SGPRs") if "ew_interp_kernel" in n]
    assert len(kernels) == 30 and all(k == 0 for n, k in kernels if not n.startswith("_ZN3ocn16ew_interp_kernelILi14ELb1E")), kernels


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_fused_kernels_of_wide_elements_keep_their_registers(tmp_path):
    """Too many vectors in flight spill complex sums in the row form; several column forms in one kernel spill
    counts of comparisons."""
    src = tmp_path / "fused.hip"
    rows = [("B_ADD", "DT_C32", "DT_C32"), ("B_MUL", "DT_C32", "DT_C32"), ("B_MUL", "DT_C64", "DT_C64"), ("B_SUB", "DT_C64", "DT_C64"),
            ("B_ABSGT", "DT_C32", "DT_BOOL"), ("B_MUL", "DT_F32", "DT_F32"), ("B_MUL", "DT_F16", "DT_F16")]
    cols = [("B_MUL", "DT_F32", "DT_F32", 0), ("B_MUL", "DT_F32", "DT_F32", 2), ("B_MUL", "DT_C64", "DT_C64", 1), ("B_EQ", "DT_F32", "DT_BOOL", 0),
            ("B_GT", "DT_F64", "DT_BOOL", 1), ("B_EQ", "DT_C32", "DT_BOOL", 2), ("B_ABSGT", "DT_C32", "DT_BOOL", 0)]
    src.write_text("".join(f'#include "{os.path.join(CSRC, h)}"\n' for h in ("fred_kernels.hpp", "red_launch.hpp")) + "namespace ocn {\n" + "".join(
        f"template __global__ void fred_rows_lean_kernel<Sig<{op}, {t}, {t}, {o}, 2>, R_SUM>(const RedLeanArgs);\n" for op, t, o in rows) + "".join(
        f"template __global__ void fred_cols_kernel<Sig<{op}, {t}, {t}, {o}, 2>, R_SUM, {bc}, false>(const RedArgs);\n" for op, t, o, bc in cols) + "}\n")
    kernels = _spills(src, "VGPRs")
    assert len(kernels) == len(rows) + len(cols) and all(k == 0 for _, k in kernels), kernels
