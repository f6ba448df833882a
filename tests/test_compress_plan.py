"""How the one-pass compressor's workgroups share out their blocks, replayed on the host (compress_pass_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_block_has_one_owner_however_workgroups_start(tmp_path):
    exe = str(tmp_path / "compress_pass")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-pthread",
                    "-I", os.path.join(ROOT, "paper_2406_11674_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "compress_pass_driver.cpp")], check=True)
    out = subprocess.run([exe, "3000"], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout
