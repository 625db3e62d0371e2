"""Where the bf16 attention kernels take their bias from: the window of diagonals is chosen only where its LDS leaves a compute
unit as many workgroups as the slice does, for every distance of the last bucket, length and form, and dk/dv with 64 channels
always has two.  Host code only."""
import os
import shutil
import subprocess

import pytest

import paper_2203_17189_amd as P

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_workgroups_per_unit(tmp_path):
    exe, lib = str(tmp_path / "attention_plan"), os.path.dirname(os.path.abspath(P.__file__))
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-x", "hip",
                        os.path.join(HERE, "attention_plan", "driver.cpp"), "-o", exe, "-L", lib, "-l:libt5mi.so",
                        f"-Wl,-rpath,{lib}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-1000:]
