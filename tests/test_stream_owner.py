"""Which thread's stream hipStreamPerThread means, host logic only: a C++ check compiled against
the built library (tests/owner_check.cpp)."""
import os
import shutil
import subprocess

import pytest

from tests.conftest import ROOT

PKG = os.path.join(ROOT, "paper_2502_06155_amd")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_each_thread_owns_its_per_thread_stream(tmp_path):
    if not os.path.exists(os.path.join(PKG, "libtileattn.so")):
        pytest.skip("library not built")
    exe = tmp_path / "owner_check"
    cmd = ["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "owner_check.cpp"), "-o", str(exe), "-L", PKG, "-ltileattn",
           f"-Wl,-rpath,{PKG}"]
    rocm_lib = "/opt/rocm/lib"
    if os.path.isdir(rocm_lib):
        cmd += ["-L", rocm_lib, "-lamdhip64", f"-Wl,-rpath,{rocm_lib}"]
    subprocess.run(cmd, check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and "stream owners ok" in res.stdout, res.stdout + res.stderr
