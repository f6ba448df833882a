"""How the one-pass compressor's workgroups share out their blocks, replayed on the host (compress_pass_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def _run(tmp_path, calls, flags):
    exe = str(tmp_path / "compress_pass")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-pthread", *flags,
                    "-I", os.path.join(ROOT, "paper_2406_11674_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "compress_pass_driver.cpp")], check=True)
    out = subprocess.run([exe, str(calls)], capture_output=True, text=True, timeout=120,
                         env=dict(os.environ, LD_PRELOAD="", TSAN_OPTIONS="halt_on_error=1"))
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr


def test_every_block_has_one_owner_however_workgroups_start(tmp_path):
    _run(tmp_path, 3000, ["-O2"])


def test_what_waves_read_of_each_other_has_been_given_out(tmp_path):
    _run(tmp_path, 200, ["-O1", "-g", "-fsanitize=thread"])
