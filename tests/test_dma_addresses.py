"""Addresses of the loads that write LDS, at sizes no other test reaches: the
wide form of operands of 2 GiB and more (an FP64 G_K from c = 16384 on), leading
dimensions up to their bound, ragged tiles.  Host code only: the header's
own address functions against 64-bit addresses (tests/host_dma/addresses.cpp)."""
import os
import re
import subprocess

import pytest

from paper_1708_04539_amd.build import CSRC, HIPCC

HERE = os.path.dirname(os.path.abspath(__file__))


def test_dma_addresses(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "addresses")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1", "-w",
                        "-I", CSRC, os.path.join(HERE, "host_dma", "addresses.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    last = re.fullmatch(r"mismatches (\d+), narrow (\d+), wide (\d+)", r.stdout.splitlines()[-1])
    assert r.returncode == 0 and last and last.group(1) == "0", r.stdout[-3000:]
    assert int(last.group(2)) > 100 and int(last.group(3)) > 50
