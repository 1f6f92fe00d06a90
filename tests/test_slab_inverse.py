"""The slab tests' inverse direction is a correctly rounded division in the kernels that answer
visibility: in the device assembly of the one-sample-per-lane density kernels no hardware
reciprocal stands but as a division's own start (no GPU needed)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_07571_amd", "csrc")
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")


def test_reciprocals_belong_to_divisions(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not installed")
    out = tmp_path / "k_density.s"
    r = subprocess.run([HIPCC, "-O3", "--offload-arch=gfx950", "-std=c++17", "-ffp-contract=off", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        "-x", "hip", "--offload-device-only", "-S", os.path.join(CSRC, "k_density.hip"), "-o", str(out)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    kernel, count = None, {}
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\S+):", line)
        if m:
            kernel = m.group(1)
        for op in ("v_rcp_f32", "v_div_fixup_f32"):
            if op in line:
                count[(kernel, op)] = count.get((kernel, op), 0) + 1
    walks = {k for k, _ in count if re.search(r"k_densityILi1ELi1ELb[01]ELb0E", k or "")}
    assert len(walks) == 2, walks
    for k in walks:
        assert count[(k, "v_rcp_f32")] <= count[(k, "v_div_fixup_f32")], (k, count)
