"""What entry points launch, recorded on the host by a stand-in for the runtime (no GPU code, no GPU needed), and the order
of a kernel's work, with the settings of the build that csrc/common.hpp admits."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def check(name, tmp_path, flags):
    obj, exe = str(tmp_path / "check.o"), str(tmp_path / "check")
    subprocess.run([HIPCC, "--cuda-host-only", "-x", "hip", "-O1", "-fPIC", "-I" + os.path.join(ROOT, "paper_2107_01499_amd", "csrc"),
                    "-I" + os.path.join(ROOT, "include"), "-c", os.path.join(ROOT, "tests", "host", name + "_check.hip"), "-o", obj] + flags, check=True)
    subprocess.run([os.environ.get("CXX", "g++"), obj, "-o", exe], check=True)   # without the runtime's library
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert res.stdout.startswith("OK ")


@pytest.mark.parametrize("rows", [2, 4])
def test_topk_compression(tmp_path, rows):
    check("topk_launches", tmp_path, ["-DBAGUA_RPW_TOPK=%d" % rows])


def test_optimizer_steps_after_topk(tmp_path):
    check("optim_launches", tmp_path, [])


def test_every_worker_of_a_sign_server_step_is_in_a_group(tmp_path):
    check("sign_groups", tmp_path, [])


def test_rounds_in_low_precision(tmp_path):
    check("ring_launches", tmp_path, [])


@pytest.mark.parametrize("rows", [2, 4])
def test_averages_and_gathers(tmp_path, rows):
    check("fused_launches", tmp_path, ["-DBAGUA_RPW_COMPRESS=%d" % rows, "-DBAGUA_RPW_SIGN=%d" % rows])
