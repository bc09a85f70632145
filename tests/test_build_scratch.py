"""Registers of the kernels on big tiles: a workgroup of 1024 threads has 128 per lane, and what does
not fit goes to scratch memory on every worker's turn.  Compiles for gfx950 without a GPU."""
import os
import re
import subprocess

from paper_1910_00643_amd import build


def test_big_tiles_use_no_scratch(tmp_path):
    flags = [f for f in build.FLAGS if f != "-shared"]
    r = subprocess.run([build.hipcc(), *flags, "--cuda-device-only", "-c", "-x", "hip",
                        "-Rpass-analysis=kernel-resource-usage",
                        os.path.join(build.CSRC, "slowmo_kernels.hip"), "-o", str(tmp_path / "k.o")],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr
    scratch = {}
    for line in r.stderr.splitlines():
        if m := re.search(r"Function Name: (\S+)", line):
            name = m.group(1)
        elif m := re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line):
            scratch[name] = int(m.group(1))
    # k_local_outer_big<BASE, BF16, FIRST, POLICY, VPT>; policy 1 runs only where a test asks for it
    big = {n: v for n, v in scratch.items()
           if "k_outer_big" in n or ("k_local_outer_big" in n and re.search(r"Li0ELi1[246]E", n))}
    assert len(big) == 3 + 8 * 3, sorted(big)
    assert not {n: v for n, v in big.items() if v}
