"""Workspace sizes on the host: a layer of either value type can be created from
the size that ffsl_workspace_bytes gives without the type, and from its typed
size, and from no less.  The device queries are answered by the driver
(workspace_driver.cpp), so no GPU is needed and nothing is launched."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_layers_fit_the_workspace_they_ask_for(tmp_path):
    from paper_2411_03171_amd import _build
    if not os.path.exists(_build.LIB):
        pytest.skip("libffsl.so not built (run __graft_entry__.build())")
    exe = str(tmp_path / "workspace_driver")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(ROOT, "tests", "workspace_driver.cpp"),
                           _build.LIB, "-Wl,-rpath," + os.path.dirname(_build.LIB), "-Wl,--export-dynamic",
                           "-L" + rocm + "/lib", "-Wl,-rpath," + rocm + "/lib", "-lamdhip64"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr
    assert "0 failures" in r.stdout
