"""The asynchronous attention kernels meet at plain s_barrier instructions and let the next tile overwrite the LDS slot that
was read before it, so no LDS read may still be on its way when a wave arrives there.  Checked on the compiled kernels:
every ds_read ahead of an s_barrier, in program order, is covered by an lgkmcnt wait."""
import os
import re
import subprocess

import pytest

from paper_2508_11661_amd import build as B


def test_no_lds_read_in_flight_at_a_barrier(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "attn.s")
    subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, "attn.hip"), "-o", out], check=True,
                   capture_output=True)
    text = open(out).read()
    seen = 0
    for m in re.finditer(r"^(_ZN\S*dma\S*):.*?\n(.*?)\.Lfunc_end\d+:", text, re.M | re.S):
        in_flight = barriers = 0
        for line in m[2].split("\n"):
            op = line.strip()
            if op.startswith("ds_"):
                in_flight += 1
            elif op.startswith("s_waitcnt"):
                wait = re.search(r"lgkmcnt\((\d+)\)", op)
                in_flight = min(in_flight, int(wait[1])) if wait else in_flight
            elif op.startswith("s_barrier"):
                barriers += 1
                assert in_flight == 0, f"{m[1]}: {in_flight} LDS accesses in flight at barrier {barriers}"
        seen += barriers > 1
    assert seen >= 4
