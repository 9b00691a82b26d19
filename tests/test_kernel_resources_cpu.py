"""Registers of the compiled kernels, read from the metadata of the library that the build made, and the compile-time
choice of rows per wave.  A kernel body that is rewritten without a change of meaning can still lose a workgroup per CU, or spill."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2107_01499_amd", "lib", "libbagua_hip.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LLVM = os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{symbol of the kernel: (VGPRs, scratch bytes per lane)}"""
    d = tmp_path_factory.mktemp("codeobjects")
    fat, co = str(d / "fatbin"), str(d / "co")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, LIB, os.devnull], check=True)
    with open(fat, "rb") as f:
        data = f.read()
    found = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):     # one bundle per source file
        at = m.start() + 32
        for _ in range(struct.unpack_from("<Q", data, m.start() + 24)[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + name]
            at += 24 + name
            if b"gfx950" not in target or not size:
                continue
            with open(co, "wb") as f:
                f.write(data[m.start() + offset:m.start() + offset + size])
            notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", co], capture_output=True, text=True, check=True).stdout
            for block in notes.split("  - .agpr_count:")[1:]:
                found[re.search(r"\.symbol:\s+(\S+)", block)[1]] = tuple(
                    int(re.search(r"\.%s:\s+(\d+)" % key, block)[1]) for key in ("vgpr_count", "private_segment_fixed_size"))
    return found


def test_no_kernel_uses_scratch_memory(kernels):
    assert len(kernels) > 100
    assert [n for n, v in kernels.items() if v[1]] == []


@pytest.mark.parametrize("family", ["k_ring_avg_lpILi1ELi2E", "k_ring_avg_lpILi2ELi2E", "k_peer_avg_lpILi2E"])
def test_small_rings_and_pairs_run_at_full_occupancy(kernels, family):
    """64 VGPRs are eight waves per SIMD, four workgroups of 4096-element chunks per CU; with 66 it is three."""
    of = {n: v[0] for n, v in kernels.items() if family in n}
    assert of and max(of.values()) <= 64, of


@pytest.mark.parametrize("knob", ["COMPRESS", "DRR", "SIGN", "DRR_SIGN", "TOPK", "DRR_TOPK", "LP"])
def test_rows_per_wave_without_a_kernel_instance_do_not_build(knob):
    src = os.path.join(ROOT, "paper_2107_01499_amd", "csrc", "api.hip")
    cmd = [HIPCC, "--cuda-host-only", "-fsyntax-only", "-I" + os.path.dirname(src), "-I" + os.path.join(ROOT, "include"), src]
    res = subprocess.run(cmd + ["-DBAGUA_RPW_%s=8" % knob], capture_output=True, text=True)
    assert res.returncode != 0 and "no kernel instance" in res.stderr
