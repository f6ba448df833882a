"""How the vector products share out their work: LDS, items and columns of every plan, on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_plans_of_the_vector_products(tmp_path):
    exe = tmp_path / "gemv_plan_driver"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                           "-I", os.path.join(ROOT, "paper_2406_11674_amd", "csrc"),
                           os.path.join(ROOT, "tests", "gemv_plan_driver.cpp"), "-o", str(exe)])
    proc = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout
    assert proc.stdout.startswith("ok"), proc.stdout
