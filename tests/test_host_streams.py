"""Streams and events of the stage schedule, without a GPU:
tests/sanitize/stream_check.cpp runs the library's host code against a stand-in
for the HIP runtime (fake_hip.cpp) that models streams as queues, under
AddressSanitizer and UndefinedBehaviorSanitizer, and the host-thread scenario
under ThreadSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2206_04959_amd", "csrc")
SAN = os.path.join(ROOT, "tests", "sanitize")


def _build(tmp, *sanitize):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the ROCm headers")
    exe = str(tmp / "stream_check")
    cmd = [gxx, "-std=c++17", "-O1", "-g", *sanitize, "-fno-omit-frame-pointer", "-D__HIP_PLATFORM_AMD__",
           "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(CSRC, "stage.cpp"),
           *(os.path.join(SAN, f) for f in ("stream_check.cpp", "fake_hip.cpp", "fake_launch.cpp")),
           "-pthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.fixture(scope="module")
def checked(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("streams"), "-fsanitize=address,undefined", "-fno-sanitize-recover=all")


def _run(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert f"{scenario} passed" in r.stdout


@pytest.mark.parametrize("scenario", ["lifetime", "moved", "captured", "threads", "many_pairs", "failed_create"])
def test_stage_streams(checked, scenario):
    _run(checked, scenario)


def test_stage_streams_from_threads_race_free(tmp_path):
    exe = _build(tmp_path, "-fsanitize=thread")
    r = subprocess.run([exe, "failed_create"], capture_output=True, text=True, timeout=60)
    if "unexpected memory mapping" in r.stderr:
        pytest.skip("ThreadSanitizer does not run on this kernel's address layout")
    _run(exe, "threads")
