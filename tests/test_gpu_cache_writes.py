"""GPU: the cache-writing kernels at the edges of their shapes -- e4m3 appends eight elements a lane (head sizes, blocks that take
several rounds to rewrite, odd head counts) and element by element, copies in pieces of 4 KiB.  Everything is bits."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import kv_update as ku
from oracle import layout as ol

pytestmark = pytest.mark.gpu


def _case(w):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase
    return GpuCase(w)


@pytest.mark.parametrize("d,block,heads,aligned", [(128, 16, 8, True), (128, 64, 3, True), (64, 32, 1, True), (256, 64, 2, True),
                                                   (128, 32, 2, False)])
def test_append_e4m3(d, block, heads, aligned):
    from paper_2602_12029_amd.runtime import to_device
    geo = wl.Geometry(2 * heads, heads, d, block, "bf16", "fp8_e4m3")
    w = wl.make_workload("app", geo, 2, [20, 1], [[0, 1], [1]], [0, block - 2, 3], pool_factor=6.0, seed=d + block)
    case = _case(w)
    for step in range(block + 5):
        k, v = w.step_tokens(step)
        dev = []
        for x in (k, v):
            t = to_device(x, "bf16")
            if not aligned:                                       # two bytes past a 16-byte boundary
                room = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
                room[1:].copy_(t.view(-1))
                t = room[1:].view(t.shape)
            dev.append(t)
        dest = case.batch.append_step(case.pool, *dev)
        odest = ol.append_step(case.opool, case.olay, None)
        assert np.array_equal(dest, odest)
        for r in range(w.num_requests):
            ku.append_token(case.data.kv, case.data.scales, "fp8_e4m3", odest[r], k[r], v[r])
        torch.cuda.synchronize()
        assert np.array_equal(case.batch.kv.cpu().numpy(), case.data.kv), step
        assert np.array_equal(case.batch.scales.cpu().numpy().view(np.int32), case.data.scales.view(np.int32)), step
    case.close()


# blocks of several pieces, of a piece and a bit, of less than one; enough pieces for four a wave, and a count that four do
# not divide; launches past the size from which an ingest keeps its loads apart; tiles of 2 KiB and less; rows of 9 and 5 chunks
@pytest.mark.parametrize("geo,tokens", [((16, 2, 128, 64, "bf16", "bf16"), [700, 65]), ((8, 4, 256, 16, "f32", "f32"), [33, 100]),
                                        ((4, 2, 64, 48, "f32", "f32"), [100, 47]), ((4, 2, 64, 16, "bf16", "bf16"), [40, 3]),
                                        ((4, 1, 128, 16, "bf16", "bf16"), [16 * 8193 + 5]), ((8, 4, 128, 64, "bf16", "fp8_e4m3"), [500, 3]),
                                        ((4, 1, 128, 16, "bf16", "bf16"), [16 * 16384 + 5, 33]), ((4, 1, 128, 32, "f32", "f32"), [32 * 4100 + 9]),
                                        ((8, 4, 128, 16, "bf16", "fp8_e4m3"), [500, 3]), ((8, 4, 64, 16, "bf16", "fp8_e4m3"), [90, 16]),
                                        ((4, 2, 72, 48, "bf16", "bf16"), [100, 3]), ((4, 2, 20, 16, "f32", "f32"), [40, 16])])
def test_copies_in_pieces(geo, tokens):
    """Ingest, staging out and in: the image holds every block of the tables in order, and comes back into other blocks."""
    from paper_2602_12029_amd import binding as B
    from paper_2602_12029_amd.runtime import DecodeBatch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hq, h, d, block, qd, kvd = geo
    g = B.geometry(*geo)
    n = len(tokens)
    ids = np.arange(n, dtype=np.int32)
    need = sum(-(-t // block) for t in tokens)
    order = np.random.default_rng(3).permutation(need + 5).astype(np.int32)
    pool = B.ps_pool_create(need + 5, order)
    lay = B.ps_kv_layout(pool, g, tokens, ids, ids * 0, ids * 0)
    kv_t = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8_e4m3": torch.uint8}[kvd]
    src_t = torch.float32 if kvd == "f32" else torch.bfloat16
    kv = torch.zeros((need + 5, h, 2, block, d), dtype=kv_t, device="cuda")
    scales = torch.zeros((need + 5, h, 2), device="cuda") if kvd == "fp8_e4m3" else None
    batch = DecodeBatch(lay, g, n, torch.zeros((n, hq, d), dtype=torch.float32 if qd == "f32" else torch.bfloat16, device="cuda"), kv, scales)
    gen = torch.Generator(device="cuda").manual_seed(1)
    k, v = (torch.randn((sum(tokens), h, d), device="cuda", generator=gen).to(src_t) for _ in range(2))
    batch.kv_ingest(0, k, v)
    table = B.ps_layout_tables(lay, n, n)["prefix_blk"].astype(np.int64)
    torch.cuda.synchronize()
    if kvd != "fp8_e4m3":
        at = tok = 0
        for t in tokens:
            blocks = torch.from_numpy(table[at:at + -(-t // block)]).cuda()
            for which, src in enumerate((k, v)):
                got = kv[blocks, :, which].permute(0, 2, 1, 3).reshape(-1, h, d)
                assert torch.equal(got[:t], src[tok:tok + t]) and not got[t:].any()
            at += -(-t // block)
            tok += t
    _, scales_off, total = B.ps_stage_layout(lay)
    image = torch.zeros(total, dtype=torch.uint8, device="cuda")
    batch.stage_out(image)
    torch.cuda.synchronize()
    want = kv[torch.from_numpy(table).cuda()].contiguous().view(-1).view(torch.uint8)
    assert torch.equal(image[:want.numel()], want)
    if scales is not None:
        want_s = scales[torch.from_numpy(table).cuda()].contiguous().view(-1).view(torch.uint8)
        assert torch.equal(image[scales_off:scales_off + want_s.numel()], want_s)
    batch.park(pool)
    hole = B.ps_kv_layout(pool, g, [3 * block], [0], [0], [0])       # the blocks come back in another order
    kv.zero_()
    batch.resume(pool)
    batch.stage_in(image)
    torch.cuda.synchronize()
    after = B.ps_layout_tables(lay, n, n)["prefix_blk"].astype(np.int64)
    assert not np.array_equal(after, table)
    assert torch.equal(kv[torch.from_numpy(after).cuda()].contiguous().view(-1).view(torch.uint8), want)
    for l in (lay, hole):
        B.ps_layout_release(pool, l)
    B.ps_pool_destroy(pool)
