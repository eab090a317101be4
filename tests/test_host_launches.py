"""What the library launches, looked at on the CPU: tests/_host_probe.py over a HIP runtime that notes launches and runs nothing."""
import os
import subprocess
import sys

import pytest

from paper_2011_10170_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not os.path.exists(B.LIB_PATH):
        from paper_2011_10170_amd import build
        build.build()
    out = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-I/opt/rocm/include", "-o", out, os.path.join(ROOT, "tests", "_hip_stub.c"), "-l:libstdc++.so.6"], check=True)
    return out


@pytest.mark.parametrize("check", ["wgrad_lds", "wgrad_lds_narrow", "thin_planes", "changing_counts", "alignment", "noalloc_first_layer", "no_host_memory", "no_room", "no_room_first_layer", "wgrad_choice", "wgrad_few_choice", "f32_wgrad_choice", "group_choice", "conv_choice", "f32_conv_choice"])
def test_host_side(stub, check):
    r = subprocess.run([sys.executable, "-m", "tests._host_probe", stub, check], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr


def test_kernels_chosen_for_a_network_are_remembered(tmp_path):
    exe = str(tmp_path / "choice_table")
    subprocess.run(["hipcc" if not os.path.exists("/opt/rocm/bin/hipcc") else "/opt/rocm/bin/hipcc", "--cuda-host-only", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2011_10170_amd", "csrc"), "-o", exe, os.path.join(ROOT, "tests", "choice_table.hip")],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    assert out.split("\n")[:3] == ["0 0"] * 3, out
