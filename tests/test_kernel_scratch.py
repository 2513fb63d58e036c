"""Every form of the subdomain-solve kernels (complex64 and complex128, 256 and 512 threads, the three coarse solves) and of the
exact local solves keeps its state in registers and LDS: compiled for gfx950 with the library's own flags, none
uses scratch memory.  A spill inside a step loop waits for every factor load in flight."""

import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("source,kernel,forms", [("inner_kernels.hip", "inner_solve", 12), ("direct_kernels.hip", "direct_solve", 6)])
def test_no_scratch(tmp_path, source, kernel, forms):
    from paper_2103_17081_amd import build
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    out = tmp_path / "kernels.s"
    subprocess.run([hipcc, "-x", "hip", *build.COMMON, "--cuda-device-only", "-S",
                    os.path.join(ROOT, "paper_2103_17081_amd", "csrc", source), "-o", str(out), *build.DEVICE_FLAGS],
                   check=True, capture_output=True, timeout=900)
    text = out.read_text()
    seen = 0
    for entry in text[text.index("amdhsa.kernels:"):].split("\n  - ")[1:]:
        field = dict(re.findall(r"^\s+\.(\w+):\s+(\S+)", entry, re.M))
        if kernel in field.get("name", ""):
            seen += 1
            assert field["private_segment_fixed_size"] == "0" and field["vgpr_spill_count"] == "0", field["name"]
    assert seen == forms
