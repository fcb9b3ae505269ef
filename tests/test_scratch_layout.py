"""Scratch layouts of the library, checked on the host: what one call of a sweep writes must not overlap."""
import os
import subprocess

import paper_1707_08265_amd as d
from paper_1707_08265_amd import build as lib_build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_regions_of_a_ring_sweep_do_not_overlap(tmp_path):
    exe = str(tmp_path / "scratch_layout_check")
    lib = os.path.dirname(os.path.abspath(d.LIB_PATH))
    subprocess.check_call(["hipcc", *lib_build.FLAGS, os.path.join(HERE, "scratch_layout_check.hip"), "-o", exe,
                           "-L", lib, "-ldgn", f"-Wl,-rpath,{lib}"], stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-3000:]
    assert " 0 faults" in r.stdout
