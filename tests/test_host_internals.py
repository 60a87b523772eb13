"""Host-side internals without an entry point of their own, CPU only: small C++ programs under tests/native, compiled with
the library's host sources under AddressSanitizer and UndefinedBehaviorSanitizer."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_12029_amd", "csrc")


def test_addresses_are_numbers():
    """The calls of a serving loop take addresses as integers; text, bytes and ctypes objects are refused before the library."""
    from paper_2602_12029_amd import binding as B
    geo = B.geometry(4, 2, 64, 16, "f32", "f32")
    pool = B.ps_pool_create(8)
    layout = B.ps_kv_layout(pool, geo, [20], [0], [0], [3])
    for bad in (b"tables", "tables", ctypes.create_string_buffer(4096), ctypes.pointer(ctypes.c_int(0)), object()):
        with pytest.raises((TypeError, ValueError)):
            B.ps_layout_upload(layout, bad)
        with pytest.raises((TypeError, ValueError)):
            B.ps_merge_states(layout, 16, bad, 16)
    for none in (None, 0):
        with pytest.raises(B.PsError) as e:
            B.ps_layout_upload(layout, none)
        assert e.value.status == B.PS_ERR_INVALID_ARG
    B.ps_layout_release(pool, layout)
    B.ps_pool_destroy(pool)


@pytest.mark.parametrize("program", ["block_order", "upload_staging", "plan_builds", "solo_items", "schedule_balance", "copy_ranges", "tile_rows"])
def test_native(program, tmp_path):
    exe = str(tmp_path / program)
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(ROOT, "tests", "native", program + ".cpp"),
                    os.path.join(CSRC, "layout.cpp"), "-pthread", "-o", exe], check=True)
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert res.returncode == 0 and res.stdout.strip().endswith("ok"), res.stdout + res.stderr
