"""The host runtime's buffers without a GPU: tests/host_runtime_stub.cpp stands
in for the HIP runtime under liblbm355 and checks the buffers of every launch."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2409_16781_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    from paper_2409_16781_amd import _build

    if not os.path.exists(_build.LIB):
        _build.build()
    exe = str(tmp_path_factory.mktemp("stub") / "host_runtime_stub")
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                          "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), "-o", exe,
                          os.path.join(ROOT, "tests", "host_runtime_stub.cpp"), _build.LIB, "-Wl,-rpath," + PKG,
                          "-Wl,--allow-shlib-undefined"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return exe


@pytest.mark.parametrize("case", ["tuner_ring", "force_field_memory", "tuner_memory"])
def test_buffers_of_every_launch(stub, case):
    res = subprocess.run([stub, case], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.startswith("ok"), res.stdout + res.stderr
