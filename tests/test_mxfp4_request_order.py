"""The MXFP4 GEMM's first wait counts requests: pair 0's activations are in LDS when at most that many younger ones are
outstanding.  So the requests must be emitted in the order in which the source makes them, which the compiler is free to change
where nothing pins it: read from the assembly of this source.  Host only."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2511_10645_amd import build


def _prologues(asm):
    """per NTW: the requests in front of the first barrier (X activations to LDS, W weights, s scales), and its wait's count"""
    for m in re.finditer(r"^_ZN4paro17mxfp4_gemm_kernelILi(\d)E\S*:\s", asm, re.M):
        requests, wait = "", None
        for line in asm[m.end():].splitlines():
            line = line.strip()
            if line.startswith("buffer_load"):
                requests += "X" if line.endswith(" lds") else "W" if line.startswith("buffer_load_dwordx4") else "s"
            elif line.startswith("s_waitcnt") and "vmcnt" in line:
                wait = int(re.search(r"vmcnt\((\d+)\)", line).group(1))
            elif line.startswith("s_barrier"):
                break
        yield int(m.group(1)), requests, wait


@pytest.mark.skipif(not shutil.which(build.HIPCC), reason="no hipcc")
def test_requests_leave_in_the_order_that_the_first_wait_counts(tmp_path):
    out = str(tmp_path / "mxfp4.s")
    cmd = [build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "mxfp4.hip"), "-o", out]
    subprocess.run(cmd, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    with open(out) as f:
        found = list(_prologues(f.read()))
    assert sorted(n for n, _, _ in found) == [1, 2]
    for ntw, requests, wait in found:
        scales, weights = "s" * (1 + 2 * ntw), "W" * (2 * ntw)
        assert requests == scales + ("XXXX" + weights) * 3 + scales, (ntw, requests)
        assert wait == 8 * ntw
        assert len(requests) - (requests.index("XXXX") + 4) >= wait, (ntw, requests, wait)
