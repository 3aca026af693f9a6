"""Register budgets of the built kernels, read from the library's metadata."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1909_02894_amd", "libdirac.so")
LLVM = "/opt/rocm/lib/llvm/bin"


@pytest.mark.skipif(not (os.path.exists(LLVM + "/llvm-readelf") and os.path.exists(LIB)),
                    reason="needs the built library and llvm-readelf")
def test_two_batch_workgroups_share_a_compute_unit(tmp_path):
    # 256 threads are one wave on each SIMD: up to 256 of its 512 registers let a second
    # workgroup in
    shutil.copy(LIB, tmp_path / "libdirac.so")
    subprocess.run([LLVM + "/llvm-objdump", "--offloading", "libdirac.so"], cwd=tmp_path, check=True,
                   capture_output=True)
    used = {}
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" in f:
            notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", f], cwd=tmp_path, check=True, capture_output=True,
                                   text=True).stdout
            for k in notes.split("- .agpr_count:")[1:]:
                name = re.search(r"\.name:\s+(\S+)", k).group(1)
                if "batch_group_kernel" in name:
                    used[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1))
    assert len(used) >= 2 * 2 * 8
    assert max(used.values()) <= 256, {k: v for k, v in used.items() if v > 256}
