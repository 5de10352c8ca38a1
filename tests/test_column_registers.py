"""Registers of the one-block solver's kernels: its vectors live in them, and an
array that the compiler keeps as one tuple is spilled as a whole where it does
not fit (an iteration then takes ten times as long).  Compiles the kernels for
the GPU's architecture; needs no GPU."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.slow
@pytest.mark.parametrize("source,kernels", [("column.hip", 30), ("column_pre.hip", 14)])
def test_no_vector_is_spilled(tmp_path, source, kernels):
    from paper_2310_11222_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    asm = tmp_path / "kernels.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source),
                    "-o", str(asm)], check=True, capture_output=True, text=True)
    seen = {}
    for m in re.finditer(r"\.amdhsa_kernel (\S*k_column\S*)(.*?)\.end_amdhsa_kernel", asm.read_text(), re.S):
        seen[m.group(1)] = int(re.search(r"private_segment_fixed_size (\d+)", m.group(2)).group(1))
    assert len(seen) >= kernels
    # a few values of a thread may wait in memory; a vector of 8 doubles or 32 floats may not
    assert max(seen.values()) <= 512, {k: v for k, v in seen.items() if v > 512}
