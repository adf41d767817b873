"""Registers of the bf16 forward, from the compiler's resource report (CPU): what its item loops keep in scratch memory.

A reload waits for everything in flight, tile requests and output stores among it, so a few spilled registers show in the run
time of every item.  The instances without a mask have one kind of item and none; those with one have two kinds, whose
operands must not live through each other's pairs (33 and 32 registers when they did).  The limits leave the compiler a few."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def spills(source):
    """{kernel name with its template arguments: vector registers spilled}"""
    from paper_2007_14062_amd.build import CSRC, HIPCC_FLAGS

    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    log = subprocess.run([hipcc, *flags, "-w", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--offload-device-only", "-S", "-o",
                          os.devnull, "-Rpass-analysis=kernel-resource-usage", os.path.join(CSRC, source)],
                         capture_output=True, text=True, check=True).stderr
    out, name = {}, None
    for line in log.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            t = re.match(r"_ZN2bb\d+([a-z_0-9]+?)I((?:L[ib]\d+E)+)E", m.group(1))
            name = t and (t.group(1), tuple(map(int, re.findall(r"L[ib](\d+)E", t.group(2)))))
        m = re.search(r"VGPRs Spill: (\d+)", line)
        if m and name:
            out[name] = int(m.group(1))
    return out


def test_bf16_forward():
    got = spills("fwd_bf16.hip")
    assert len(got) == 12, got
    plain, masked, options, drop = range(4)
    most = {plain: 0, masked: 8, options: 8, drop: 8}
    for (kernel, args), n in got.items():
        assert n <= (0 if kernel == "fwd_rows_bf16" else most[args[0]]), (kernel, args, n)
