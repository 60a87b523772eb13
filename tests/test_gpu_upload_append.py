"""GPU: tables and the tokens of a decode step in one launch (ps_layout_upload_append) against the two calls it stands for: the same
tables, pool and scale bits, for every format, with requests that append nothing and table sizes on both sides of the range that
a kernel moves."""
import numpy as np
import pytest
import torch

from paper_2602_12029_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv,d,heads", [("f32", 64, (4, 2)), ("bf16", 128, (28, 4)), ("fp8_e4m3", 128, (8, 3)), ("fp8_e4m3", 256, (8, 4)), ("fp8_e4m3", 96, (2, 1))])
@pytest.mark.parametrize("prompts,tokens,kernel_sized", [(3, 40, False), (20, 1000, True)])
def test_one_launch_stores_what_two_do(kv, d, heads, prompts, tokens, kernel_sized):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h, block = heads[1], 16
    q_heads = heads[0] - heads[0] % h
    geo = B.geometry(q_heads, h, d, block, "f32" if kv == "f32" else "bf16", kv)
    requests = 2 * prompts
    req_prompt, model = np.repeat(np.arange(prompts, dtype=np.int32), 2), np.tile(np.arange(2, dtype=np.int32), prompts)
    suffix = (np.arange(requests) * 5 % 33).astype(np.int32)
    blocks = prompts * -(-tokens // block) + int((-(-suffix // block)).sum()) + requests
    gen = torch.Generator(device="cuda").manual_seed(prompts + d)
    esz = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8_e4m3": torch.uint8}[kv]
    pool_bits = torch.randint(0, 120, (blocks, h, 2, block, d), device="cuda", generator=gen).to(esz)
    scales = (torch.rand((blocks, h, 2), device="cuda", generator=gen) / 200 + 1e-4) if kv == "fp8_e4m3" else None
    t = torch.float32 if kv == "f32" else torch.bfloat16
    steps = [[(torch.randn((requests, h, d), device="cuda", generator=gen) * 2.0 ** i).to(t) for _ in range(2)] for i in range(3)]
    active = (np.arange(requests) % 4 != 1).astype(np.int32)
    stream = int(torch.cuda.current_stream().cuda_stream)
    results = []
    for fused in (False, True):
        pool = B.ps_pool_create(blocks)
        lay = B.ps_kv_layout(pool, geo, np.full(prompts, tokens, np.int32), req_prompt, model, suffix)
        data, sc = pool_bits.clone(), scales.clone() if scales is not None else None
        for new_k, new_v in steps:
            B.ps_layout_append(pool, lay, requests, active)
            size = B.ps_layout_device_bytes(lay)
            assert ((16 << 10) < size <= (1 << 20)) == kernel_sized
            tables = torch.zeros(size, dtype=torch.uint8, device="cuda")
            where = (tables.data_ptr(), new_k.data_ptr(), new_v.data_ptr(), data.data_ptr(), sc.data_ptr() if sc is not None else 0, stream)
            if fused:
                B.ps_layout_upload_append(lay, *where)
            else:
                B.ps_layout_upload(lay, tables.data_ptr(), stream)
                B.ps_kv_append(lay, *where)
        torch.cuda.synchronize()
        results.append((tables, data.view(torch.uint8), sc.view(torch.int32) if sc is not None else tables))
        if fused:
            for bad in ((where[0], 0, *where[2:]), (0, *where[1:])):
                with pytest.raises(B.PsError) as e:
                    B.ps_layout_upload_append(lay, *bad)
                assert e.value.status == B.PS_ERR_INVALID_ARG
        torch.cuda.synchronize()
        B.ps_layout_release(pool, lay)
        B.ps_pool_destroy(pool)
    for a, b in zip(*results):
        assert torch.equal(a, b)
    assert not torch.equal(results[0][1], pool_bits.view(torch.uint8))


@pytest.mark.parametrize("kv,d,heads", [("bf16", 64, (32, 32)), ("f32", 64, (33, 33)), ("bf16", 128, (5, 5)), ("bf16", 64, (1, 1))])
def test_a_wave_per_row_of_a_token(kv, d, heads):
    """Tokens of 2 to 66 rows, four to a workgroup: a last one that is full, half full, and the only one."""
    test_one_launch_stores_what_two_do(kv, d, heads, 20, 1000, True)
