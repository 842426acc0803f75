"""The time-sliced finder's window loop at the end of the largest calls it
takes (2^31 - 1 hits), on the CPU: hough_tw.h itself, a thread per lane."""
import os
import shutil
import subprocess

import pytest

from paper_2511_02742_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path_factory.mktemp("tw") / "tw_last_hits"
    # -fwrapv: integers wrap as they do on the device
    subprocess.check_call([gxx, "-std=c++20", "-O1", "-fwrapv", "-pthread", "-w", "-I", os.path.join(HERE, "native", "lanes"),
                           "-I", os.path.join(build.CSRC, "..", "..", "include"), "-I", build.CSRC,
                           os.path.join(HERE, "native", "tw_last_hits.cpp"), "-o", str(exe)])
    return str(exe)


@pytest.mark.parametrize("hits", [40, 200, 400])
@pytest.mark.parametrize("end", [500, 2**31 - 2000, 2**31 - 64, 2**31 - 1])
def test_windows_at_the_last_hits(program, end, hits):
    r = subprocess.run([program, str(end), str(hits)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    assert r.stdout.startswith("ok")
