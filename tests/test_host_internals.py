"""Host-side internals without an entry point of their own, CPU only: small C++ programs under tests/native, compiled with
the library's host sources under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_12029_amd", "csrc")


@pytest.mark.parametrize("program", ["block_order", "upload_staging"])
def test_native(program, tmp_path):
    exe = str(tmp_path / program)
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(ROOT, "tests", "native", program + ".cpp"),
                    os.path.join(CSRC, "layout.cpp"), "-pthread", "-o", exe], check=True)
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert res.returncode == 0 and res.stdout.strip().endswith("ok"), res.stdout + res.stderr
