"""`xg2_matcher_accept_tokens` beside a fill that is still running, on the CPU: `api.cpp` with the HIP runtime and the kernels replaced
by a device whose fills end when the host waits for them (`hostcheck/accept_beside_main.cpp`), under AddressSanitizer and
UndefinedBehaviorSanitizer."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2601_04426_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("accept_beside") / "accept_beside_main")
    cmd = ["g++", "-O0", "-std=c++17", "-pthread", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wno-subobject-linkage",
           "-I/opt/rocm/include", "-D__HIP_PLATFORM_AMD__", "-o", out, os.path.join(HERE, "hostcheck", "accept_beside_main.cpp"),
           os.path.join(CSRC, "grammar.cpp"), os.path.join(CSRC, "tables.cpp")]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
    return out


@pytest.mark.parametrize("mode", ["allocations", "statuses", "threads"])
def test_accept_beside_a_fill(exe, mode):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:alloc_dealloc_mismatch=0")
    env.pop("LD_PRELOAD", None)
    res = subprocess.run([exe, mode], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env, timeout=120)
    assert res.returncode == 0 and res.stdout.startswith("ok"), res.stdout[-3000:]
