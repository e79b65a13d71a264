"""Host rules of the workspaces, built on their own: how the wide branches'
scratch is cut (csrc/branchplan.h), over random plans, and how a workspace
grows (csrc/workspace.h), against a device with little memory and under
capture."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["branchplan_check", "workspace_check"])
def test_native(tmp_path, name):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path / name)
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I" + os.path.join(ROOT, "paper_2604_15380_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", name + ".cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([out], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
