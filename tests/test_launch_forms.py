"""Which form a step's launch takes, on the CPU: the library's host code compiled against a stand-in for the HIP
runtime (tests/native/host_runtime), its launches recorded, under AddressSanitizer + UndefinedBehaviorSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("launch_forms") / "launch_forms_host")
    native = os.path.join(ROOT, "tests", "native")
    subprocess.check_call(["g++", "-std=c++17", "-w", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-fno-omit-frame-pointer", "-I", os.path.join(native, "host_runtime"), os.path.join(native, "launch_forms_host.cpp"),
                           os.path.join(ROOT, "paper_2603_13358_amd", "csrc", "ppd_plan.cpp"), "-pthread", "-o", path])
    return path


@pytest.mark.parametrize("what", ["merged_once", "four_waves", "second_round", "on_waves", "estimate", "pipelined", "by_block", "modes_share_a_plan"])
def test_decode_only_launch_forms(exe, what):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0")
    env.pop("LD_PRELOAD", None)
    res = subprocess.run([exe, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env, timeout=120)
    assert res.returncode == 0 and "ok" in res.stdout, res.stdout[-3000:]
