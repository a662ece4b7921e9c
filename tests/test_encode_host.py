"""The host half of zs_encode_device against a stand-in for the HIP runtime (tests/hip_double.cpp), without a GPU: calls that
the runtime lets down fall back to a copy or are refused, and no slot of pinned memory is lost by it."""
import os
import subprocess

import pytest

from paper_2603_17435_amd import build as zs_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = tmp_path_factory.mktemp("hip_double")
    packer, double, exe = out / "packer.o", out / "double.o", out / "program"
    common = list(zs_build.COMMON)

    def run(cmd):
        return subprocess.run([str(c) for c in cmd], check=True, capture_output=True, text=True).stdout
    run([zs_build.HIPCC, "-c", "--cuda-host-only", "--offload-arch=gfx950", os.path.join(zs_build.CSRC, "zs_encode_device.hip"), "-o", packer] + common)
    run([zs_build.HIPCC, "-x", "c++", "-c", os.path.join(HERE, "hip_double.cpp"), "-o", double, "-pthread",
         "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include"] + common)
    run([zs_build.HIPCC, "-x", "c++", "-c", os.path.join(zs_build.CSRC, "zs_encode.cpp"), "-o", out / "bound.o", "-pthread"] + common)
    # the kernels' code, which is not there and not needed
    device_code = [w.split()[-1] for w in run(["nm", packer]).splitlines() if "__hip_fatbin_" in w]
    run(["g++", "-o", exe, packer, double, out / "bound.o", "-pthread"] + [f"-Wl,--defsym={s}=0" for s in device_code])
    return exe


@pytest.mark.parametrize("scenario", ["plain", "no_pinned_memory", "no_mapping", "threads", "failed_wait", "failed_launch",
                                      "failed_launch no_pinned_memory", "capture"])
def test_packer_host_code(program, scenario):
    done = subprocess.run([str(program)] + scenario.split(), capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout + done.stderr
