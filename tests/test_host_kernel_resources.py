"""Compiled kernels (no GPU): the registers that decide how many workgroups of the
small-launch hop and of the 5D kernel a CU holds; how the FP16 hop at Ls = 2 loads its links."""
import pathlib
import re
import subprocess

import pytest

from paper_1804_08593_amd import build

# a workgroup of the small-launch hop is 8 waves, two on each of a CU's 4 SIMDs of 512
# VGPRs (allocated in eights): n workgroups fit up to 512 / (2 n) VGPRs
WORKGROUPS = {("F64", 6): 2, ("F64", 8): 2, ("F64", 12): 2, ("F64", 16): 2, ("F64", 20): 2,
              ("F32", 16): 3, ("F32", 20): 3, ("F32", 24): 3}


def _listing(tmp_path, header, kernels):
    src = tmp_path / "k.hip"
    src.write_text(f'#include "{header}"\nnamespace mspcg {{\n' +
                   "".join(f"template __global__ void {k};\n" for k in kernels) + "}\n")
    r = subprocess.run(["hipcc", *build.CXXFLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", str(src),
                        "-o", str(tmp_path / "k.s")], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    return (tmp_path / "k.s").read_text()


def _vgprs(tmp_path, cases):
    text = _listing(tmp_path, "hop_small.h",
                    [f"hop_small_kernel<{p}, {ls}, true, {cg}>(HopArgs<{p}>)"
                     for p, ls in cases for cg in ("true", "false")])
    out = {}
    name = None
    for ln in text.splitlines():
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


def test_fived_kernel_keeps_its_residency(tmp_path):
    """The 5D kernel's LDS lets a CU hold six workgroups of four waves in FP32 and FP16:
    where the s-vector of a thread leaves them the room, its registers do too."""
    build_dir = pathlib.Path(build.CSRC)
    r = subprocess.run(["hipcc", *build.CXXFLAGS, "-I", build.CSRC, "--cuda-device-only", "-S",
                        str(build_dir / "blas.hip"), "-o", str(tmp_path / "b.s")],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    v, name = {}, None
    for ln in (tmp_path / "b.s").read_text().splitlines():
        m = re.match(r"\s*\.amdhsa_kernel \S*fived_kernelINS_3(F\d\d)ELi(\d+)E", ln)
        if m:
            name = (m[1], int(m[2]))
        m = re.match(r"\s*\.amdhsa_next_free_vgpr (\d+)", ln)
        if m and name:
            v[name] = int(m[1])
        if ".end_amdhsa_kernel" in ln:
            name = None
    for prec in ("F32", "F16"):
        for ls in (2, 4, 6, 8, 16):
            assert v[prec, ls] <= 512 // 6 // 8 * 8, (prec, ls, v)


def test_fp16_hop_loads_unstaged_links_in_wide_loads(tmp_path):
    """At Ls = 2 the links do not fit in LDS beside each other and every thread loads its
    72 entries: the two directions of a mu in five loads, not 4 bytes at a time."""
    text = _listing(tmp_path, "hop_impl.h",
                    ["hop_kernel<F16, 2, false, false, false, false>(HopArgs<F16>)"])
    loads = re.findall(r"\b(global|flat)_load_(\w+)", text)
    single = sum(w in ("dword", "ushort", "short_d16", "short_d16_hi") for _, w in loads)
    assert single <= 16, single  # scales and arguments
    assert len(loads) <= 64, len(loads)
