"""GPU: the float32-probability kernel of the PS_VARIANT_WAVE family on the matrix cores, at the edges of its tiles.

Every pair of formats and head size, blocks of 16, 48 and 64 tokens, segments that end at, before and after a 16- and a
32-token tile, row groups on both sides of 16, 32 and 64 rows, masked rows, other pool layouts, infinite values, and
the pools it does not take (blocks that are no multiple of 16 tokens, misaligned base pointers: the vector kernel).

Bars: float32 outputs 1e-5 max-abs / 1e-5 relative RMS (sums of up to a few hundred float32 terms: some 10 ulp of 1);
bf16 outputs are the float32 result rounded once, relative error at most 2^-9 per element, 1.7e-3 relative RMS over
uniformly distributed mantissas; held at 2e-3 relative RMS and 2^-8 of the largest output."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import errors
from oracle import attention as oa

pytestmark = pytest.mark.gpu

PREFIX = [1, 15, 16, 33, 300]
SUFFIX = [0, 1, 16, 17, 31, 32, 33, 47, 64, 65, 127, 128, 129, 2, 5, 250, 63, 80]


def _workload(geo, models, seed=3, prefix=PREFIX):
    membership = [list(range(m)) for m in models]
    n = sum(models)
    return wl.make_workload("tile", geo, max(models), prefix, membership, [SUFFIX[i % len(SUFFIX)] for i in range(n)],
                            pool_factor=1.3, seed=seed)


def _case(w, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase
    return GpuCase(w, **kw)


def _check(case, visible=None):
    from paper_2602_12029_amd.runtime import from_device
    g = case.w.geometry
    ref, ref_lse = oa.decode_attention(case.q_bits, g.q_dtype, case.data.kv, case.data.scales, g.kv_dtype, case.olay, None, visible)
    torch.cuda.synchronize()
    got, lse = from_device(case.batch.out), from_device(case.batch.lse)
    max_abs, rel_rms, _ = errors(got, ref)
    print(f"max_abs={max_abs:.2e} rel_rms={rel_rms:.2e}", flush=True)
    assert np.isfinite(got).all()
    if g.q_dtype == "f32":
        assert max_abs <= 1e-5 and rel_rms <= 1e-5
    else:
        assert max_abs <= np.abs(ref).max() * 2.0 ** -8 and rel_rms <= 2e-3
    seen = np.isfinite(ref_lse)
    assert np.array_equal(np.isneginf(lse), ~seen)
    assert np.abs(lse[seen] - ref_lse[seen]).max(initial=0.0) <= 1e-5


def _step(case, visible=None):
    case.poison_workspace()
    case.batch.decode_attention()
    _check(case, visible)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("kv,q", [("f32", "f32"), ("bf16", "bf16"), ("fp8_e4m3", "bf16"), ("bf16", "f32"), ("f32", "bf16"),
                                  ("fp8_e4m3", "f32")])
def test_formats_heads_and_row_groups(kv, q, d):
    """Row groups of 4, 16, 20, 36 and 68 rows per KV head; whole-segment chunks, chunks of one and of three tiles."""
    geo = wl.Geometry(8, 2, d, 16, q, kv)
    case = _case(_workload(geo, [1, 4, 5, 9, 17]))
    for pc, sc in ((0, 0), (32, 32), (96, 64)):
        case.replan(pc, sc, "wave", "wave")
        _step(case)
    case.close()


@pytest.mark.parametrize("block", [8, 16, 48, 64])
@pytest.mark.parametrize("kv,q,d", [("f32", "f32", 64), ("bf16", "bf16", 64), ("fp8_e4m3", "bf16", 128)])
def test_block_sizes_and_visible_lengths(kv, q, d, block):
    geo = wl.Geometry(4, 2, d, block, q, kv)
    w = _workload(geo, [2, 9, 1, 3, 20])
    case = _case(w)
    _step(case) if d == 64 else None
    full = w.prefix_len[w.req_prompt]
    visible = np.random.default_rng(5).integers(0, full + 1)
    visible[:3] = [0, full[1], 0]
    for pc in (0, 96):
        case.replan(pc, 0, "wave", "wave")
        case.set_visible(visible)
        _step(case, visible)
    case.close()


@pytest.mark.parametrize("layout", ["token_major", "planes"])
@pytest.mark.parametrize("kv,q,d", [("f32", "f32", 128), ("bf16", "bf16", 256), ("fp8_e4m3", "bf16", 64)])
def test_pool_layouts(kv, q, d, layout):
    case = _case(_workload(wl.Geometry(8, 2, d, 32, q, kv), [1, 5, 2, 1, 4]), pool_layout=layout)
    _step(case)
    case.close()


@pytest.mark.parametrize("kv,q", [("f32", "f32"), ("bf16", "bf16"), ("fp8_e4m3", "bf16")])
def test_planes_far_apart(kv, q):
    """K and V planes more than 2 GiB apart: past the matrix-core decode kernel's offsets, so the plan takes this family."""
    from paper_2602_12029_amd import binding as B
    from paper_2602_12029_amd.runtime import DecodeBatch
    geo = wl.Geometry(8, 2, 128, 16, q, kv)
    case = _case(_workload(geo, [1, 5, 2, 1, 4]), pool_layout="planes")
    w, near = case.w, case.batch.kv
    plane = near[0].numel()
    far = (1 << 31) // near.element_size() + 4096 + plane
    flat = torch.zeros(far + plane, dtype=near.dtype, device="cuda")
    flat[:plane] = near[0].reshape(-1)
    flat[far:] = near[1].reshape(-1)
    wide = B.geometry(8, 2, 128, 16, q, kv, (2 * 16 * 128, 16 * 128, far, 128))
    pool = B.ps_pool_create(w.num_blocks, w.free_order)
    layout = B.ps_kv_layout(pool, wide, w.prefix_len, w.req_prompt, w.req_model, w.suffix_len)
    assert B.ps_layout_plan(layout, w.num_requests)["prefix_variant"] == B.PS_VARIANT_WAVE
    case.batch = DecodeBatch(layout, wide, w.num_requests, case.batch.q, flat, case.batch.scales)
    _step(case)
    case.close()
    B.ps_layout_release(pool, layout)
    B.ps_pool_destroy(pool)


def test_cache_policies_and_misaligned_pool():
    """Streamed and cacheable loads give the same bits; a pool that starts off a 16-byte boundary is served too."""
    from paper_2602_12029_amd import binding as B
    case = _case(_workload(wl.Geometry(8, 2, 64, 16, "f32", "f32"), [1, 5, 2, 1, 18]))
    outs = []
    for policy in (B.PS_KV_POLICY_STREAM, B.PS_KV_POLICY_CACHEABLE):
        case.replan(kv_cache_policy=policy)
        _step(case)
        outs.append(case.batch.out.clone())
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))
    flat = torch.zeros(case.batch.kv.numel() + 4, device="cuda")
    case.batch.kv = flat[1:1 + case.batch.kv.numel()].view(case.batch.kv.shape).copy_(case.batch.kv)
    assert case.batch.kv.data_ptr() % 16 == 4
    _step(case)
    case.close()


@pytest.mark.parametrize("kv,q", [("f32", "f32"), ("bf16", "bf16")])
def test_infinite_values(kv, q):
    """An infinite element of V comes out as that infinity for the requests that see it, and nowhere else."""
    w = _workload(wl.Geometry(8, 2, 64, 16, q, kv), [2, 4, 1, 5, 3])
    case = _case(w)
    t = case.olay
    at = {0: (0, float("inf")), 3: (7, float("-inf")), 4: (299, float("inf"))}    # prompt -> (token, value)
    for p, (tok, value) in at.items():
        blk = int(t.prefix_blk[t.prefix_blk_indptr[p] + tok // 16])
        case.batch.kv[blk, 1, 1, tok % 16, 5] = value
    case.poison_workspace()
    case.batch.decode_attention()
    torch.cuda.synchronize()
    got = case.batch.out.float().cpu().numpy()
    want = np.zeros(got.shape)
    for r in range(w.num_requests):
        if int(w.req_prompt[r]) in at:
            want[r, 4:, 5] = at[int(w.req_prompt[r])][1]
    assert np.array_equal(np.where(np.isinf(got), got, 0.0), want)
    assert not np.isnan(got).any()
    case.close()


@pytest.mark.parametrize("block", [8, 16, 32])
@pytest.mark.parametrize("q,d", [("bf16", 64), ("bf16", 128), ("f32", 128), ("f32", 256)])
def test_scales_of_a_callers_own_quantiser(q, d, block):
    """e4m3 tiles whose K or V scale is zero (a tile of zeros by amax / 448) or negative, in segments that end inside a tile and
    under visible lengths; the same bars as above, since the oracle multiplies by the same scales."""
    w = _workload(wl.Geometry(4, 2, d, block, q, "fp8_e4m3"), [2, 9, 1, 3, 5])
    case = _case(w)
    sc = case.data.scales
    pick = np.random.default_rng(17).integers(0, 4, sc.shape)
    sc[:] = np.where(pick == 0, 0.0, np.where(pick == 1, -sc, sc)).astype(np.float32)
    case.batch.scales.copy_(torch.from_numpy(sc))
    case.replan(0, 0, "wave", "wave")
    _step(case)
    visible = np.random.default_rng(5).integers(0, w.prefix_len[w.req_prompt] + 1)
    case.set_visible(visible)
    _step(case, visible)
    case.close()
