"""Register counts that decide how many workgroups a CU holds, read from the
compiled kernels (host only: compiled to gfx950 assembly, nothing runs)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_04875_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_fp8_append_keeps_five_workgroups_a_cu(tmp_path):
    """Four-wave workgroups put one wave on each SIMD: five fit its 512
    registers at up to 96 each (allocated in eights), four at 103."""
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path / "kv_pool.s"
    subprocess.run([HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", "-x", "hip",
                    "--cuda-device-only", "-S", os.path.join(CSRC, "kv_pool.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    counts = {}
    for block in out.read_text().split("  - .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        counts[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1))
    fp8 = {k: v for k, v in counts.items() if "append_kernelIth" in k}     # bf16 in, codes out
    assert len(fp8) == 12, sorted(counts)
    assert max(fp8.values()) <= 96, fp8
