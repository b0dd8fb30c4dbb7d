"""Generated-code check of k_sort.hip (CPU): the scatter's lanes exchange places in LDS behind fences."""
import os
import re
import subprocess

from paper_2004_11127_amd import build as kbuild


def test_scatter_orders_its_lanes_accesses(tmp_path):
    """Each of the eight rounds reads a digit's place, moves it on and reads it again in the next round,
    from other lanes of the wave: a barrier of the schedule alone would not order the accesses."""
    out = str(tmp_path / "sort.ll")
    cmd = [kbuild.HIPCC] + kbuild.flags_for("k_sort.hip") + [
        "--cuda-device-only", "-S", "-emit-llvm", os.path.join(kbuild.CSRC, "k_sort.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        body = re.search(r"define [^\n]*sort_scatter_kernel.*?\n}\n", f.read(), re.S).group(0)
    fences = len(re.findall(r'fence syncscope\("wavefront(?:-one-as)?"\) acq_rel', body))
    barriers = body.count("call void @llvm.amdgcn.wave.barrier()")
    assert fences >= barriers > 0 and barriers % 2 == 0
