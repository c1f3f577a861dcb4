"""No kernel spills a register for part of its lanes only.

Where lanes come back together, the compiler (LLVM of ROCm 7.2) can place the spill
of a register in front of the instruction that brings them back. The lanes that
did not take the branch then keep what the scratch memory held, with no error.
The kernels that are held to many waves a SIMD spill a lot; one that fell into
this found no neighbours.
"""
import concurrent.futures as cf
import glob
import os
import re
import subprocess

import pytest

from paper_2003_10850_amd import build


def early_spills(path):
    r = subprocess.run([build.hipcc(), *build.FLAGS, "--cuda-device-only", "-S", path, "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return scan(r.stdout)


def scan(text):
    found, kernel, spills, start = [], "", [], False
    for line in text.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            kernel, start = m.group(1), False
        if re.match(r"\.LBB\d+_\d+:|; %bb", line):
            spills, start = [], True  # a block begins
        t = line.strip()
        if not start or not t or t[0] in ";.":
            continue
        if "scratch_store" in t and "Spill" in t:
            spills.append(t)
        elif re.match(r"s_or_b64 exec, exec,", t):  # the lanes come back together
            found += [(kernel, s) for s in spills]
            start = False
        elif re.match(r"s_\w*(saveexec|branch)|s_\w+_b64 exec,", t):
            start = False
    return found


def test_the_scan_sees_one():
    text = """_Zk:
.LBB7_47:
\tscratch_store_dwordx2 off, v[18:19], off offset:108 ; 8-byte Folded Spill
\ts_or_b64 exec, exec, s[22:23]
.LBB7_48:
\ts_or_b64 exec, exec, s[20:21]
\tscratch_store_dword off, v1, off offset:4 ; 4-byte Folded Spill
"""
    assert [k for k, _ in scan(text)] == ["_Zk"]


def test_no_kernel_spills_before_its_lanes_are_back():
    srcs = sorted(glob.glob(os.path.join(build.CSRC, "*.hip")))
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        for src, found in zip(srcs, ex.map(early_spills, srcs)):
            assert not found, (os.path.basename(src), found[:4])
