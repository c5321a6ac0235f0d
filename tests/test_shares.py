"""How units are dealt out to the eight XCDs, host logic only: a C++ check compiled against
the built library (tests/share_check.cpp)."""
import os
import re
import shutil
import subprocess

import pytest

from tests.conftest import ROOT

PKG = os.path.join(ROOT, "paper_2502_06155_amd")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_shares_hold_equal_work(tmp_path):
    if not os.path.exists(os.path.join(PKG, "libtileattn.so")):
        pytest.skip("library not built")
    exe = tmp_path / "share_check"
    cmd = ["g++", "-std=c++17", "-O1", "-I", os.path.join(PKG, "csrc"), "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "share_check.cpp"), "-o", str(exe), "-L", PKG, "-ltileattn",
           f"-Wl,-rpath,{PKG}"]
    rocm_lib = "/opt/rocm/lib"
    if os.path.isdir(rocm_lib):
        cmd += ["-L", rocm_lib, "-lamdhip64", f"-Wl,-rpath,{rocm_lib}"]
    subprocess.run(cmd, check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    print(res.stdout)
    assert res.returncode == 0, res.stdout + res.stderr
    got = {m.group(1): (int(m.group(2)), float(m.group(3)))
           for m in re.finditer(r"^(\S+) equal (\d) most (\S+)$", res.stdout, re.M)}
    assert len(got) == 10
    assert got["uniform"][0] == 1
    for name in ("mixed-fwd", "mixed-bwd", "share-sym"):
        assert got[name][0] == 0 and got[name][1] < 1.02, name
    cut = {n: (int(u), int(w)) for n, u, w in
           re.findall(r"^(cut-\S+) cut (\d+) units by work (\d)$", res.stdout, re.M)}
    assert len(cut) == 5
    for name in ("cut-d96", "cut-batch", "cut-d128"):
        assert cut[name][0] > 0 and cut[name][1] == 0, name
    assert cut["cut-none"] == (0, 1)
    every = dict(re.findall(r"^(every-\S+) every call work (\d)$", res.stdout, re.M))
    assert every == {"every-share": "1", "every-long": "1", "every-short": "0"}
    # the cut by work is taken only where it makes the launch shorter
    choice = {m.group(1): tuple(float(m.group(i)) for i in (2, 3, 4))
              for m in re.finditer(r"^(choice-\S+) counts (\S+) work (\S+) chosen (\S+)$", res.stdout, re.M)}
    assert len(choice) == 8
    for name in ("choice-sym4", "choice-fwd", "choice-d128", "choice-tail"):
        counts, work, chosen = choice[name]
        assert work > counts == chosen, name
    for name in ("choice-share-heads", "choice-many"):
        counts, work, chosen = choice[name]
        assert chosen == work < counts, name
    assert choice["choice-share-sym"][2] <= choice["choice-share-sym"][0]
