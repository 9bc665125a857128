"""The library's host side, CPU only: tests/c/host_driver.cpp runs libaqs.so on
a stand-in for the HIP runtime whose streams work only when somebody waits for
them, one scenario per run (see the program's header)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2507_20802_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libaqs.so")):
        pytest.skip("libaqs.so is not built")
    hipcc = os.environ.get("HIPCC") or shutil.which("hipcc") or os.path.join(ROCM, "bin", "hipcc")
    exe = str(tmp_path_factory.mktemp("host_driver") / "host_driver")
    obj = exe + ".o"
    for cmd in ([hipcc, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-fPIE",
                 "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                 "-c", os.path.join(ROOT, "tests", "c", "host_driver.cpp"), "-o", obj],
                # the program's symbols come before the runtime's, which it does not name
                [shutil.which("g++") or "g++", "-rdynamic", obj, "-o", exe, "-L", PKG, "-laqs",
                 f"-Wl,-rpath,{PKG}", f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}", "-Wl,--allow-shlib-undefined"]):
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
    return exe


@pytest.mark.parametrize("scenario", ["linear_start_polls", "linear_start_polls_profiled", "slot_loads_wait",
                                      "side_stream_joins", "side_stream_joins_destroy",
                                      "length_plain", "length_extrapolated", "length_linear",
                                      "length_round", "length_live", "staging_without_pinned_memory",
                                      "failed_writes_are_not_believed"])
def test_scenario(driver, scenario):
    res = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip().endswith("ok"), res.stdout + res.stderr
