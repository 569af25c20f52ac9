"""The solve server sets no request up with graphs, whatever its options say: on
the host build of the server, with a set-up that refuses them.  No GPU is used."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2605_04335_amd", "csrc")
STUB = os.path.join(HERE, "server_host")


def test_requests_are_set_up_without_graphs(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path / "drive_graphs")
    cmd = [gxx, "-std=c++17", "-O1", "-I", STUB, "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    for s in (os.path.join(CSRC, "server.hip"), os.path.join(CSRC, "memory.hip"), os.path.join(CSRC, "capi.hip"),
              os.path.join(STUB, "graphs.cpp"), os.path.join(STUB, "drive.cpp")):
        cmd += ["-x", "c++", s]
    r = subprocess.run(cmd + ["-o", out, "-lpthread"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([out, "200", "2000", "64", "8"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "done 200 failed 0" in r.stdout, r.stdout
