"""What the compiler makes of the device code, read from the assembly and the
resource remarks of a build for gfx950 (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2511_02742_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """hough_kernels.hip: (assembly lines per function, resource remarks per kernel)."""
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / "k.s"
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
           os.path.join(build.CSRC, "hough_kernels.hip"), "-S", "-o", str(out), "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    code = {}
    for m in re.finditer(r"^(_Z\S+):.*?(?=^\.Lfunc_end)", out.read_text(), re.M | re.S):
        lines = [x.split(";")[0].strip() for x in m[0].splitlines()[1:]]
        code[m[1]] = [x for x in lines if x]
    remarks = {blk.split()[0]: blk for blk in re.split(r"remark: Function Name: ", r.stderr)[1:]}
    return code, remarks


VMEM = re.compile(r"(global|flat|buffer|scratch)_")
STORES_IN = re.compile(r"s_waitcnt vmcnt\(0\)")


@pytest.mark.parametrize("kind", ["k_find", "k_argmax", "find_event_call"])
def test_a_returned_slot_is_written_back_whole(kernels, kind):
    """A large event's slot goes from one workgroup to the next (on another
    XCD, behind another L2) by a flag that one thread clears. Before it does, every
    wave has waited for its own stores (ahead of the barrier) and the thread
    for its write-back of the L2."""
    code, _ = kernels
    seen = 0
    for name, lines in code.items():
        if kind not in name:
            continue
        for i, line in enumerate(lines):
            if not line.startswith("buffer_wbl2"):
                continue
            seen += 1
            flag = next(k for k in range(i + 1, len(lines)) if VMEM.match(lines[k]))
            assert "atomic_swap" in lines[flag], (name, lines[flag])
            assert any(STORES_IN.match(x) for x in lines[i + 1:flag]), (name, lines[i - 3:flag + 1])
            bar = max(k for k in range(i) if lines[k] == "s_barrier")
            wait = max(k for k in range(bar) if STORES_IN.match(lines[k]))
            assert bar - wait <= 8 and not any(VMEM.match(x) for x in lines[wait:bar]), (name, lines[bar - 8:bar + 1])
    assert seen >= 9   # three ways out of an event, three workgroup sizes


def _remark(remarks, kind, what):
    return {n: int(re.search(what + r": (\d+)", blk).group(1)) for n, blk in remarks.items() if kind in n}


def test_finder_kernels_keep_no_scratch(kernels):
    """The largest-bin search and the first of two shapes, like the finder, keep
    their working set in registers and LDS; where the event function is a call (the
    time-sliced finder, the list of events) it saves some 20 to 50 registers."""
    _, remarks = kernels
    for kind, sizes in (("k_argmax", 3), ("k_picked", 6)):
        scratch = _remark(remarks, kind, r"ScratchSize \[bytes/lane\]")
        assert len(scratch) == sizes and set(scratch.values()) == {0}, scratch
    for kind, sizes in (("k_tw_run", 6), ("k_list", 2)):
        scratch = _remark(remarks, kind, r"ScratchSize \[bytes/lane\]")
        assert len(scratch) == sizes and max(scratch.values()) <= 192, scratch


def test_finder_kernels_share_a_cu_alike(kernels):
    """Every kernel that takes large-event slots runs four waves per SIMD (at most
    128 registers), so none has more workgroups resident than another."""
    _, remarks = kernels
    for kind in ("k_find", "k_argmax", "k_picked", "k_list", "k_tw_run"):
        waves = _remark(remarks, kind, r"Occupancy \[waves/SIMD\]")
        assert len(waves) >= 2 and set(waves.values()) == {4}, waves
