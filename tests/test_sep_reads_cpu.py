"""The separable kernels read only records that the slope pass writes.

tests/native/sep_reads.cpp builds plans of many shapes with the library's own
plan builder (discs, balls and boxes on grids whose spacings differ by up to
eight, short periodic axes, every class of footprints) and checks each column
that the kernels read, the weightless ones past a footprint included, against
the instance's reachable box.  CPU only: no kernel runs."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_separable_reads_stay_in_the_reachable_box(tmp_path):
    from paper_2104_14561_amd import build as B
    try:
        hipcc = B.hipcc()
    except RuntimeError as e:
        pytest.skip(str(e))
    names = [name for _, name, _ in B.units() if name != "fk_host"]
    objs = [os.path.join(B.HERE, "_build", n + ".o") for n in names]
    if not all(os.path.exists(o) for o in objs):
        B.build()
    exe = str(tmp_path / "sep_reads")
    obj = exe + ".o"
    subprocess.check_call([hipcc, "-x", "hip"] + B.compile_flags() +
                          ["-c", os.path.join(ROOT, "tests", "native", "sep_reads.cpp"), "-o", obj])
    subprocess.check_call([hipcc, f"--offload-arch={B.ARCH}", "-o", exe, obj] + objs)
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
