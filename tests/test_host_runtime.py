"""The host runtime past its first device call, under sanitizers and without a
GPU: ``svf_runtime.cpp`` with HIP and the kernel launchers replaced by host
functions (``native/host_runtime_main.cpp``).  Address and undefined-behaviour
sanitizers for every mode, the thread sanitizer for those that start threads."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
SOURCES = [os.path.join(ROOT, "paper_2606_22327_amd", "csrc", "svf_runtime.cpp"),
           os.path.join(HERE, "native", "host_runtime_main.cpp")]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def build(directory, sanitizer):
    exe = os.path.join(str(directory), "host_runtime")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-pthread", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.dirname(SOURCES[0]), f"-fsanitize={sanitizer}",
                           "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", *SOURCES, "-o", exe])
    return exe


@pytest.fixture(scope="module")
def address(tmp_path_factory):
    return build(tmp_path_factory.mktemp("address"), "address,undefined")


@pytest.fixture(scope="module")
def threads(tmp_path_factory):
    return build(tmp_path_factory.mktemp("thread"), "thread")


def run(exe, mode):
    env = {k: v for k, v in os.environ.items() if not k.startswith("SVFSIM_")}
    r = subprocess.run([exe, mode], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"{mode}: exit {r.returncode}\n{r.stdout[-2000:]}\n{r.stderr[-4000:]}"
    assert "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, r.stderr[-4000:]
    assert f"{mode}: ok" in r.stdout


@pytest.mark.parametrize("mode", ["reset", "rings", "reads", "device", "whole", "validate"])
def test_under_address_and_undefined_sanitizers(address, mode):
    run(address, mode)


@pytest.mark.parametrize("mode", ["reads", "validate"])
def test_under_thread_sanitizer(threads, mode):
    run(threads, mode)
