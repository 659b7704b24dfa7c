"""The 256 x 256 kernel's registers, from the compiler's own listing (no GPU): every accumulator is in a register all the time, so what else spills costs it."""
import os
import re
import subprocess

from paper_2604_02525_amd import build


def test_the_large_tiles_spill_next_to_nothing():
    """Up to 62 scalars where gathered K-channels come first (kernel arguments, kept in lanes of a vector register over the tile); a store routine that
    formed the offsets of all 64 rows of a lane beforehand made them 205 and more."""
    cmd = [build.hipcc()] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm_mx.hip"), "-o", "-"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    entries = re.findall(r"- \.agpr_count:.*?\.wavefront_size", r.stdout, re.S)
    kernels = {re.search(r"\.name:\s+(\S+)", e)[1]: e for e in entries}
    tiled = {n: e for n, e in kernels.items() if "k_gemm_mx_tile256" in n}
    assert len(tiled) == 10
    for name, e in tiled.items():
        assert int(re.search(r"\.vgpr_spill_count:\s+(\d+)", e)[1]) == 0, name
        assert int(re.search(r"\.sgpr_spill_count:\s+(\d+)", e)[1]) <= 64, name
