"""Registers of compiled kernels (no GPU): what decides how many workgroups of the
small-launch hop a CU holds."""
import os
import re
import subprocess

import pytest

from paper_1804_08593_amd import build

# a workgroup of the small-launch hop is 8 waves, two on each of a CU's 4 SIMDs of 512
# VGPRs (allocated in eights): n workgroups fit up to 512 / (2 n) VGPRs
WORKGROUPS = {("F64", 6): 2, ("F64", 8): 2, ("F64", 12): 2, ("F64", 16): 2, ("F64", 20): 2,
              ("F32", 16): 3, ("F32", 20): 3, ("F32", 24): 3}


def _vgprs(tmp_path, cases):
    src = tmp_path / "k.hip"
    src.write_text('#include "hop_small.h"\nnamespace mspcg {\n' + "".join(
        f"template __global__ void hop_small_kernel<{p}, {ls}, true, {cg}>(HopArgs<{p}>);\n"
        for p, ls in cases for cg in ("true", "false")) + "}\n")
    r = subprocess.run(["hipcc", *build.CXXFLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", str(src),
                        "-o", str(tmp_path / "k.s")], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    out = {}
    name = None
    for ln in (tmp_path / "k.s").read_text().splitlines():
        m = re.match(r"\s*\.amdhsa_kernel \S*hop_small_kernelINS_3(F\d\d)ELi(\d+)ELb1ELb([01])E", ln)
        if m:
            name = (m[1], int(m[2]), m[3] == "1")
        m = re.match(r"\s*\.amdhsa_next_free_vgpr (\d+)", ln)
        if m and name:
            out[name] = int(m[1])
    return out


@pytest.mark.parametrize("prec", ["F64", "F32"])
def test_small_hop_with_fused_update_keeps_its_residency(tmp_path, prec):
    cases = [k for k in WORKGROUPS if k[0] == prec]
    v = _vgprs(tmp_path, cases)
    assert len(v) == 2 * len(cases)
    for k in cases:
        room = 512 // (2 * WORKGROUPS[k]) // 8 * 8
        assert v[(*k, False)] <= room and v[(*k, True)] <= room, (k, v)
