"""Index arithmetic that kernels share with the host (plain constant expressions in csrc/*.h), checked at the ends of what the
entry points accept, where a run would take many gigabytes or where a stray read would go unseen."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2505_03803_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("name", ["proxy_ranges_check", "mid_tiles_check"])
def test_index_arithmetic(name, tmp_path):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, "-o", exe, os.path.join(HERE, "host", name + ".cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.endswith(" bad 0\n"), out.stdout + out.stderr
