"""Host check (no GPU) of how the library orders its blocks of device memory:
the scenarios of host/stream_order_worker.py, each in a child process with a
HIP runtime preloaded whose streams run their work as late as they may
(host/fake_hip.cpp)."""
import os
import subprocess
import sys

import pytest

from paper_1808_10804_amd import _lib, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    lib = os.path.dirname(_lib.LIB_PATH)
    out = str(tmp_path_factory.mktemp("fake_hip") / "fake_hip.so")
    cmd = ["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", os.path.join(HOST, "fake_hip.cpp"),
           "-I", os.path.join(ROOT, "paper_1808_10804_amd", "csrc"), "-I", os.path.join(build.ROCM, "include"),
           "-L" + lib, "-l:" + os.path.basename(_lib.LIB_PATH), "-Wl,-rpath," + lib, "-o", out]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    return out


@pytest.mark.parametrize("scenario", [
    "su2_double_layer", "su2_move", "pool_waits_for_the_release", "pool_waits_for_the_mark", "pool_outlives_its_streams",
    "ring_beside_a_capture", "ring_after_a_failed_wait", "ring_after_a_destroyed_stream", "new_plan_beside_another_thread",
    "tables_outlive_their_readers", "tables_are_given_back"])
def test_stream_order(runtime, scenario):
    _run(runtime, scenario)


def _run(runtime, scenario):
    env = dict(os.environ, SYMTEN_AUTOTUNE="0", PYTHONPATH=ROOT)
    env["LD_PRELOAD"] = " ".join(p for p in (runtime, env.get("LD_PRELOAD", "")) if p)
    r = subprocess.run([sys.executable, os.path.join(HOST, "stream_order_worker.py"), scenario], cwd=ROOT, env=env,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:]


def test_eigensolver_capacity(runtime):
    """The orders and sides that the library's own eigensolver takes."""
    _run(runtime, "eigensolver_capacity")
