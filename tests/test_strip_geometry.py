"""Strips on the host (no GPU): a sweep over lengths, offsets, cascades and strip
lengths holds every cut to what the strip kernels assume (the last strip and
strip 0 have room for their states, the run-in is covered, offsets fit 32
bits); a batch's strip length equals the one found by trying each in turn; and
batches timed both ways go the faster way."""
import os
import subprocess

from paper_2607_14054_amd import sosfilt as S
from paper_2607_14054_amd.build import HIPCC

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_cut_keeps_the_kernels_assumptions(tmp_path):
    S.lib()
    exe, libdir = str(tmp_path / "strip_geometry_check"), os.path.dirname(S.LIB_PATH)
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2",
                    os.path.join(HERE, "strip_geometry_check.cpp"), "-o", exe, "-L" + libdir, "-l:libsosfilt.so",
                    "-Wl,-rpath," + libdir], check=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
