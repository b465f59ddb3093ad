"""What the library allocates and launches is on the context's device, whatever
device is current (two_devices.cpp, which stands in for the HIP runtime)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2301_05780_amd")


def test_trainer_stays_on_its_contexts_device(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++") or not os.path.exists(os.path.join(PKG, "libpdd.so")):
        pytest.skip("g++ or the built library not available")
    exe = str(tmp_path / "two_devices")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "two_devices.cpp"), "-o", exe,
                    os.path.join(PKG, "libpdd.so"), f"-Wl,-rpath,{PKG}", f"-Wl,-rpath,{os.path.join(rocm, 'lib')}",
                    f"-Wl,-rpath-link,{os.path.join(rocm, 'lib')}"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
