"""The library's calls into the HIP runtime, seen by programs that stand in for
the runtime (host_runtime.h): devices, and the launches of captured calls."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2301_05780_amd")


def _run(tmp_path, name):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++") or not os.path.exists(os.path.join(PKG, "libpdd.so")):
        pytest.skip("g++ or the built library not available")
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe,
                    os.path.join(PKG, "libpdd.so"), f"-Wl,-rpath,{PKG}", f"-Wl,-rpath,{os.path.join(rocm, 'lib')}",
                    f"-Wl,-rpath-link,{os.path.join(rocm, 'lib')}"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    return r.stdout


def test_trainer_stays_on_its_contexts_device(tmp_path):
    _run(tmp_path, "two_devices")


def test_launches_of_captured_training(tmp_path):
    """A captured batch above 1024 keeps a workgroup per 256 points, two launches a
    step (on a context that has not trained such a batch: one workgroup); up to 1024
    the four units run side by side on the waves of one workgroup, as does a single
    step up to 128 points.  Nothing is allocated in a capture."""
    got = {}
    for line in _run(tmp_path, "captured_training").splitlines():
        key, launches = line.split(":")
        got[tuple(key.split())] = launches.split()
    for batch in (32, 96, 128, 256, 1024):
        one = ["1x512"] if batch == 32 else ["1x256"]
        assert got[str(batch), "2", "captured"] == got[str(batch), "2", "fresh"] == one
    for batch, slices in ((4096, 16), (20000, 79)):
        assert got[str(batch), "2", "captured"] == [f"{slices}x256", "1x256"] * 2
        assert got[str(batch), "2", "fresh"] == ["1x512"]
    assert got["96", "1", "eager"] == got["128", "1", "eager"] == ["1x256"]
    assert got["256", "1", "eager"] == ["4x512c"]
