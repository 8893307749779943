"""How the passes' work is cut into items, on the host (CPU only): tests/host/cut_check.cpp
compares cut items with whole ones (same sources for every target, own slots, no empty item),
compiled with AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2012_06925_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not present")
def test_cut_items_meet_the_same_sources(tmp_path):
    exe = str(tmp_path / "cut_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-I" + os.path.join(ROOT, "include"), "-o", exe,
                        os.path.join(ROOT, "tests", "host", "cut_check.cpp"), os.path.join(CSRC, "tree.cpp"),
                        os.path.join(CSRC, "traverse.cpp"), "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
