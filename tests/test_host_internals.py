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


def _compile(program, where):
    exe = str(where / program)
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(ROOT, "tests", "native", program + ".cpp"),
                    os.path.join(CSRC, "layout.cpp"), "-pthread", "-o", exe], check=True)
    return exe


def _run(exe, **kw):
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env, **kw)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout.strip()


@pytest.mark.parametrize("program", ["block_order", "upload_staging", "plan_builds", "solo_items", "schedule_balance", "copy_ranges", "tile_rows"])
def test_native(program, tmp_path):
    assert _run(_compile(program, tmp_path)).endswith("ok")


def test_the_gpu_tests_of_items_a_wave_each_hold_such_items(tmp_path):
    """The plans that test_gpu_solo_items.py runs do hold short items that a wave takes alone, in the kernel they are there for."""
    import test_gpu_solo_items as gpu
    from paper_2602_12029_amd import binding as B
    exe = _compile("solo_plan", tmp_path)
    dtype = {"f32": B.PS_F32, "bf16": B.PS_BF16, "fp8_e4m3": B.PS_FP8_E4M3}
    variant = {"auto": B.PS_VARIANT_AUTO, "wave": B.PS_VARIANT_WAVE, "mfma": B.PS_VARIANT_MFMA}

    def plan(geo, cus, variants, prefix, prompt, suffix):
        words = [*geo[:4], dtype[geo[4]], dtype[geo[5]], cus, *(variant[v] for v in variants), len(prefix), len(suffix), *prefix, *prompt, *suffix]
        return [int(x) for x in _run(exe, input=" ".join(map(str, words))).split()]

    for spec in gpu.CASES + gpu.ASKED:
        w = gpu._workload(spec)
        packed, tile, _ = plan(spec[1], spec[4], (spec + ("auto",) * 2)[5:7], w.prefix_len, w.req_prompt, w.suffix_len)
        assert (tile if spec[0].startswith("tile") else packed) > 3, spec[0]
    for dtype_, models, tokens in (("bf16", 14, 36000), ("bf16", 7, 36000), ("f32", 6, 100000)):
        _, tile, spread = plan((32, 8, 64, 16, dtype_, dtype_), 8, ("auto", "auto"), [tokens - 5], [0] * models,
                               [(37 * i) % 120 + 1 for i in range(models)])
        assert tile > 3 and not spread
