"""No kernel adds products of two matrix instructions onto one accumulator.

A v_mfma_f32_16x16x16_bf16 right behind a v_mfma_f32_16x16x32_bf16 on the same
accumulator reads it before it is written: measured on the device, half of the
256 sums are wrong, and right with a wait between.  hipcc (ROCm 7.2) issues
the two back to back.  The library's own listing is checked, kernel by kernel."""
import os
import re
import subprocess

import pytest

from paper_1808_06381_amd import build


def accumulators(text):
    """{kernel: [(opcode, accumulator register range)]} of a device listing."""
    out, name = {}, None
    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name = m.group(1)
        m = re.match(r"^\s*(v_s?mfma\w*)\s+([av])\[(\d+):(\d+)\]", line)
        if m and name:
            out.setdefault(name, []).append((m.group(1), (m.group(2), m.group(3), m.group(4))))
    return out


def mixed(uses):
    seen = {}
    for op, reg in uses:
        seen.setdefault(reg, set()).add(op)
    return {reg: ops for reg, ops in seen.items() if len(ops) > 1}


def test_the_check_sees_a_mixed_kernel():
    text = ("_Zk:\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], 0\n"
            "\tv_mfma_f32_16x16x16_bf16 a[0:3], v[8:9], v[10:11], a[0:3]\n")
    assert mixed(accumulators(text)["_Zk"])


@pytest.mark.parametrize("source", [s for s in build.SOURCES if s != "sim_api.hip"])
def test_no_accumulator_is_shared(source, tmp_path):
    path = os.path.join(build.CSRC, source)
    if "_mfma_" not in open(path).read():
        return
    lst = str(tmp_path / "listing.s")
    res = subprocess.run(["hipcc", f"--offload-arch={build.ARCH}", "-O3", "-std=c++17",
                          "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", "--offload-device-only", "-S",
                          "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, path,
                          "-o", lst], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    kernels = accumulators(open(lst).read())
    assert kernels
    for name, uses in kernels.items():
        assert not mixed(uses), (name, mixed(uses))
