"""Growth of the adjoint's cached workspace against an allocator of limited
size, built with the sanitizers: a part that was refused is not asked for
again, and a workspace that will do is not given up for one that is refused."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_workspace_growth(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    driver = os.path.join(ROOT, "tests", "sanitize", "workspace_driver.cpp")
    exe = str(tmp_path / "workspace")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I" + os.path.join(ROOT, "paper_2505_22631_amd", "csrc"), driver, "-o", exe],
                   check=True, capture_output=True, text=True, timeout=300)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
