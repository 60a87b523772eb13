"""GPU: short items that a wave takes alone (four in a workgroup), in the persistent and in the tile kernel.

Batches planned for a few compute units, so that the items outnumber the workgroups; private lengths on both sides of a tile
and of the longest such item, counts that leave the last four incomplete, groups of one to sixteen rows, and lists longer
than the persistent kernel's header ring; launches over the private items alone, items that appends have made longer, beside
row groups in the form with all row tiles a wave, other pool layouts, and values that are no numbers.  (That these plans hold such
items is checked on the host, test_host_internals.py.)  Bars as everywhere (gpu_helpers), float32-probability outputs in bf16
included."""
import numpy as np
import pytest
import torch

import workloads as wl
from paper_2602_12029_amd import binding as B

pytestmark = pytest.mark.gpu

LENS = [1, 0, 16, 31, 32, 33, 64, 65, 250, 256, 257, 500, 512, 513, 17, 3, 129]

# name, (q heads, kv heads, d, block, q, kv), models, prefixes, compute units planned for
CASES = [
    ("g4", (32, 8, 128, 16, "bf16", "bf16"), 4, [700, 33, 0], 4),                 # one row tile
    ("g4_wide", (32, 8, 128, 16, "bf16", "bf16"), 8, [300, 1], 2),                # two row tiles
    ("g7_four_tiles", (28, 4, 128, 32, "bf16", "bf16"), 7, [300, 64], 1),
    ("g8_e4m3", (64, 8, 128, 16, "bf16", "fp8_e4m3"), 3, [520, 16, 40], 3),
    ("g8_two_requests", (64, 8, 128, 64, "bf16", "bf16"), 2, [90, 400, 1], 2),     # eight rows beside one row tile
    ("g1_shared_too", (8, 8, 128, 16, "bf16", "bf16"), 1, [1, 31, 32, 33, 147, 512, 513, 300, 64, 2, 90], 2),
    ("g2_e4m3_lists", (16, 8, 128, 16, "bf16", "fp8_e4m3"), 2, [40] * 30, 1),      # hundreds of items a workgroup
    ("tile_d64", (32, 8, 64, 32, "bf16", "bf16"), 4, [700, 33, 0], 2),
    ("tile_d64_wide", (16, 2, 64, 16, "bf16", "bf16"), 6, [300, 64], 1),           # G = 8, 48 rows per shared item
    ("tile_d256", (16, 4, 256, 16, "bf16", "bf16"), 5, [300, 64], 2),
    ("tile_f32_d128", (32, 8, 128, 16, "f32", "f32"), 3, [300, 64, 17], 2),
    ("tile_f32_d256", (8, 4, 256, 32, "f32", "f32"), 5, [300, 64], 1),
    ("tile_g16", (32, 2, 64, 16, "bf16", "bf16"), 3, [90, 20, 5], 1),              # sixteen rows
    ("tile_e4m3_f32", (16, 4, 64, 16, "f32", "fp8_e4m3"), 5, [90, 20], 1),
]
# the same with the kernel family of the shared and of the private segments asked for
ASKED = [
    ("tile_d128", (32, 8, 128, 16, "bf16", "bf16"), 4, [700, 33, 0], 2, "wave", "wave"),
    ("tile_d128_e4m3", (64, 8, 128, 32, "bf16", "fp8_e4m3"), 4, [700, 33, 0], 2, "wave", "wave"),
    ("tile_private", (32, 8, 128, 16, "bf16", "bf16"), 4, [700, 33, 0], 2, "mfma", "wave"),
]


def _workload(spec):
    name, geo, models, prefixes = spec[:4]
    return wl.make_workload(name, wl.Geometry(*geo), models, prefixes, [list(range(models))] * len(prefixes),
                            [LENS[i % len(LENS)] for i in range(models * len(prefixes))], pool_factor=1.3, seed=7)


def _case(spec, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase
    case = GpuCase(_workload(spec), **kw)
    case.replan(num_cus=spec[4], prefix_variant=(spec + ("auto",) * 2)[5], suffix_variant=(spec + ("auto",) * 2)[6])
    return case


def _bits(t):
    return t.view(torch.uint8)


@pytest.mark.parametrize("spec", CASES + ASKED, ids=lambda s: s[0])
def test_short_items_a_wave_each(spec):
    from gpu_helpers import check_against_oracle
    case = _case(spec)
    first = None
    for _ in range(2):
        case.poison_workspace()
        case.batch.decode_attention()
        check_against_oracle(case, label=spec[0], scaled_bar=True)
        assert not torch.isnan(case.batch.workspace_views()[1]).any()          # every partial state was written
        first = case.batch.out.clone() if first is None else first
    assert torch.equal(_bits(first), _bits(case.batch.out))
    case.close()


@pytest.mark.parametrize("spec", [c for c in CASES if c[0].startswith("tile")] + ASKED[:2], ids=lambda s: s[0])
def test_the_private_items_in_a_launch_of_their_own(spec):
    """The two passes one after the other give the bits of the one launch (the items are the same, and who takes them)."""
    case = _case(spec)
    case.poison_workspace()
    case.batch.decode_attention()
    want = case.batch.out.clone(), case.batch.lse.clone()
    case.poison_workspace()
    case.batch.prefix_attention()
    case.batch.suffix_attention()
    case.batch.merge_states()
    torch.cuda.synchronize()
    assert torch.equal(_bits(want[0]), _bits(case.batch.out)) and torch.equal(_bits(want[1]), _bits(case.batch.lse))
    case.close()


@pytest.mark.parametrize("layout", ["token_major", "planes"])
@pytest.mark.parametrize("spec", [CASES[i] for i in (0, 3, 7, 9, 10, 13)], ids=lambda s: s[0])
def test_other_pool_layouts(spec, layout):
    from gpu_helpers import check_against_oracle
    case = _case(spec, pool_layout=layout)
    case.poison_workspace()
    case.batch.decode_attention()
    check_against_oracle(case, label=f"{spec[0]} {layout}", scaled_bar=True)
    case.close()


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("spec", [CASES[i] for i in (0, 5, 7, 9, 10)], ids=lambda s: s[0])
def test_values_that_are_no_numbers(spec, value):
    """One such element of V in a private segment: it comes out for the rows of its head of that request, in its column, and
    everything else has the bits it had."""
    case = _case(spec)
    case.batch.decode_attention()
    torch.cuda.synchronize()
    want = case.batch.out.clone()
    g, t = case.w.geometry, case.olay
    group = g.num_q_heads // g.num_kv_heads
    for r in (0, 4, 7, 8):                                # segments of 1, 32, 65 and 250 tokens
        n = int(case.w.suffix_len[r])
        tok = min(n - 1, 3 * n // 4)
        blk = int(t.suffix_blk[t.suffix_blk_indptr[r] + tok // g.block_size])
        at = case.batch.kv[blk, 1, 1, tok % g.block_size]
        kept = at[5].clone()
        at[5] = value
        case.poison_workspace()
        case.batch.decode_attention()
        torch.cuda.synchronize()
        got = case.batch.out[r, group:2 * group, 5]
        assert torch.isnan(got).all() if value != value else (got == value).all()
        case.batch.out[r, group:2 * group, 5] = want[r, group:2 * group, 5]
        assert torch.equal(_bits(case.batch.out), _bits(want))
        at[5] = kept
    case.close()


def _in_64_bits(layout, w_shape, q, kv, scales):
    """Output and log-sum-exp of the layout's batch as it stands, from its tables, on the GPU in float64."""
    num_prompts, req_prompt, heads, block = w_shape
    n, q_heads, d = q.shape
    lens = B.ps_layout_lengths(layout, num_prompts, n)
    t = B.ps_layout_tables(layout, num_prompts, n)

    def segment(kind, i, length):
        ids = t[kind + "_blk"][t[kind + "_blk_indptr"][i]:t[kind + "_blk_indptr"][i + 1]].astype(np.int64)
        x = kv[torch.from_numpy(ids).cuda()]
        if scales is not None:
            x = x.view(torch.float8_e4m3fn).to(torch.float64) * scales[torch.from_numpy(ids).cuda()].double()[..., None, None]
        return x.double().permute(2, 1, 0, 3, 4).reshape(2, heads, -1, d)[:, :, :length]

    out, lse = torch.zeros(q.shape, dtype=torch.float64, device="cuda"), torch.zeros((n, q_heads), dtype=torch.float64, device="cuda")
    shared = [segment("prefix", p, int(lens["prefix_len"][p])) for p in range(num_prompts)]
    for r in range(n):
        own = segment("suffix", r, int(lens["suffix_len"][r]))
        k, v = torch.cat([shared[req_prompt[r]], own], 2)
        rows = q[r].double().reshape(heads, -1, d)
        s = torch.bmm(rows, k.transpose(1, 2).contiguous()) / d ** 0.5
        top = torch.logsumexp(s, 2)
        out[r] = torch.bmm(torch.exp(s - top[..., None]), v).reshape(q_heads, d)
        lse[r] = top.reshape(-1)
    return out, lse


def _check_in_64_bits(batch, ref, bar):
    torch.cuda.synchronize()
    err = float((batch.out.double() - ref[0]).norm() / ref[0].norm())
    lse = float((batch.lse - ref[1]).abs().max())
    print(f"rel={err:.2e} lse={lse:.2e}", flush=True)
    assert err <= bar and lse <= (1e-4 if bar <= 1e-5 else 2e-3)


@pytest.mark.parametrize("name,geo,cus", [
    ("persistent", (32, 8, 128, 16, "bf16", "bf16"), 6), ("persistent_e4m3", (64, 8, 128, 16, "bf16", "fp8_e4m3"), 6),
    ("tile_d64", (32, 8, 64, 32, "bf16", "bf16"), 8), ("tile_many", (32, 8, 64, 16, "bf16", "bf16"), 2), ("tile_f32", (16, 4, 128, 16, "f32", "f32"), 2)])
def test_items_that_appends_make_longer(name, geo, cus):
    """A turn of nine hundred tokens, one request standing still: past every limit of such an item, through the plans made anew.
    (The pool holds numbers everywhere, so the tables alone grow.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd.runtime import DecodeBatch
    q_heads, heads, d, block, q_dtype, kv_dtype = geo
    prefix, models, steps = np.array([700, 33, 260], np.int32), 4, 900
    n = models * len(prefix)
    req_prompt = np.repeat(np.arange(len(prefix)), models)
    suffix = np.arange(n) * 7 % 40
    blocks = int(sum(-(-x // block) for x in prefix)) + n * (-(-(steps + 40) // block) + 1)
    g = B.geometry(q_heads, heads, d, block, q_dtype, kv_dtype)
    pool = B.ps_pool_create(blocks, np.random.default_rng(3).permutation(blocks).astype(np.int32))
    layout = B.ps_kv_layout(pool, g, prefix, req_prompt, np.arange(n) % models, suffix)
    B.ps_layout_replan(layout, B.plan_options(0, 0, B.PS_VARIANT_AUTO, B.PS_VARIANT_AUTO, cus, 0))
    gen = torch.Generator(device="cuda").manual_seed(11)
    real = torch.randn((blocks, heads, 2, block, d), device="cuda", generator=gen)
    t, scales = torch.float32 if q_dtype == "f32" else torch.bfloat16, None
    if kv_dtype == "fp8_e4m3":
        scales = 0.01 + 0.002 * torch.rand((blocks, heads, 2), device="cuda", generator=gen)
        kv = (real / scales[..., None, None]).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    else:
        kv = real.to(t)
    q = torch.randn((n, q_heads, d), device="cuda", generator=gen).to(t)
    batch = DecodeBatch(layout, g, n, q, kv, scales)
    active = np.arange(n) != 5
    for step in range(1, steps + 1):
        B.ps_layout_append(pool, layout, n, active)
        if step in (1, 31, 90, 130, 229, 258, 500, 730, 790, steps):
            batch._sync_plan()
            batch.workspace.view(torch.float32).fill_(float("nan"))
            batch.out.fill_(float("nan"))
            batch.decode_attention()
            _check_in_64_bits(batch, _in_64_bits(layout, (len(prefix), req_prompt, heads, block), q, kv, scales),
                              1e-5 if q_dtype == "f32" else 5e-3)
    torch.cuda.synchronize()
    B.ps_layout_release(pool, layout)
    B.ps_pool_destroy(pool)


@pytest.mark.parametrize("dtype,models,tokens", [("bf16", 14, 36000), ("bf16", 7, 36000), ("f32", 6, 100000)])
def test_beside_row_groups_with_all_row_tiles_a_wave(dtype, models, tokens):
    """A batch large enough that the shared context's 24 to 56 rows go into every wave, its private segments a wave each."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd.runtime import DecodeBatch
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    suffix = np.array([(37 * i) % 120 + 1 for i in range(models)], np.int32)
    blocks = -(-tokens // 16) + 9 * models
    g = B.geometry(32, 8, 64, 16, dtype, dtype)
    pool = B.ps_pool_create(blocks, np.random.default_rng(1).permutation(blocks).astype(np.int32))
    layout = B.ps_kv_layout(pool, g, [tokens - 5], np.zeros(models, np.int32), np.arange(models), suffix)
    B.ps_layout_replan(layout, B.plan_options(0, 0, B.PS_VARIANT_AUTO, B.PS_VARIANT_AUTO, 8, 0))
    gen = torch.Generator(device="cuda").manual_seed(models)
    kv = torch.randn((blocks, 8, 2, 16, 64), device="cuda", generator=gen).to(t)
    q = torch.randn((models, 32, 64), device="cuda", generator=gen).to(t)
    batch = DecodeBatch(layout, g, models, q, kv)
    batch.out.fill_(float("nan"))
    batch.decode_attention()
    _check_in_64_bits(batch, _in_64_bits(layout, (1, np.zeros(models, int), 8, 16), q, kv, None), 1e-5 if dtype == "f32" else 2e-3)
    B.ps_layout_release(pool, layout)
    B.ps_pool_destroy(pool)
