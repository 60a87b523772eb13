"""GPU: row groups of more than 16 rows in the tile kernel -- a row tile to a wave (two or four of them, also with fewer tiles than
waves, several passes, masked rows) and, for batches large enough that the plan asks for it, all row tiles in every wave.

Bars: as in test_gpu_tile_kernel.py; the large batches against a float64 computation on the GPU with the same bars."""
import numpy as np
import pytest
import torch

import workloads as wl
from test_gpu_tile_kernel import _case, _step

pytestmark = pytest.mark.gpu


# rows per shared item = models x group (at most 64 an item): one row past a tile, two and four tiles full and not, 80 in two passes
@pytest.mark.parametrize("kv,q,d", [("bf16", "bf16", 256), ("f32", "f32", 128), ("fp8_e4m3", "f32", 64), ("bf16", "bf16", 64), ("fp8_e4m3", "bf16", 128)])
@pytest.mark.parametrize("group,models", [(17, 1), (4, 8), (3, 11), (7, 7), (4, 16), (80, 1)])
def test_a_row_tile_to_a_wave(kv, q, d, group, models):
    geo = wl.Geometry(group, 1, d, 16, q, kv)
    w = wl.make_workload("rows", geo, models, [1, 33, 300, 64, 97], [list(range(models))] * 5,
                         [(7 * i) % 40 for i in range(5 * models)], pool_factor=1.3, seed=group + models)
    case = _case(w)
    variant = "wave" if d == 128 and q == "bf16" else "auto"
    for chunk in (0, 64):
        case.replan(chunk, 0, variant, variant)
        _step(case)
    case.close()


def test_masked_rows_over_the_waves():
    """Causal chunks: every row of a wide group sees another length, some of them nothing of a chunk."""
    for kv, d, new in (("bf16", 256, 9), ("f32", 64, 30)):
        geo = wl.Geometry(8, 2, d, 16, "f32" if kv == "f32" else "bf16", kv)
        lens = [200 + new, 31 + new, new]
        w = wl.make_workload("causal", geo, new, lens, [list(range(new))] * 3, [0] * (3 * new), pool_factor=1.3, seed=d)
        case = _case(w)
        visible = np.concatenate([np.arange(n - new, n) + 1 for n in lens]).astype(np.int32)
        case.set_visible(visible)
        _step(case, visible)
        case.close()


@pytest.mark.parametrize("dtype,d,heads,group,models,tokens,variant", [
    ("bf16", 64, 8, 4, 5, 36000, 0), ("bf16", 64, 8, 4, 14, 36000, 0), ("bf16", 128, 8, 4, 7, 36000, 1), ("f32", 64, 8, 4, 6, 100000, 0)])
def test_row_tiles_in_every_wave_of_a_large_batch(dtype, d, heads, group, models, tokens, variant):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd import binding as B
    from paper_2602_12029_amd.runtime import DecodeBatch
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    geo = B.geometry(heads * group, heads, d, 16, dtype, dtype)
    n = -(-tokens // 16)
    order = np.random.default_rng(1).permutation(n).astype(np.int32)
    pool = B.ps_pool_create(n, order)
    lay = B.ps_kv_layout(pool, geo, [tokens - 5], np.zeros(models, np.int32), np.arange(models), np.zeros(models, np.int32))
    if variant:
        B.ps_layout_replan(lay, B.plan_options(0, 0, B.PS_VARIANT_WAVE, B.PS_VARIANT_WAVE))
    gen = torch.Generator(device="cuda").manual_seed(d + models)
    kv = torch.randn((n, heads, 2, 16, d), device="cuda", generator=gen).to(t)
    q = torch.randn((models, heads * group, d), device="cuda", generator=gen).to(t)
    batch = DecodeBatch(lay, geo, models, q, kv)
    batch.out.fill_(float("nan"))
    batch.decode_attention()
    torch.cuda.synchronize()
    seq = kv[torch.from_numpy(order.astype(np.int64)).cuda()].permute(2, 1, 0, 3, 4).reshape(2, heads, -1, d)[:, :, :tokens - 5]
    for h in range(heads):
        k, v = seq[0, h].double(), seq[1, h].double()
        rows = q[:, h * group:(h + 1) * group].double().reshape(-1, d)
        scores = rows @ k.t().contiguous() / d ** 0.5
        lse = torch.logsumexp(scores, 1)
        ref = torch.exp(scores - lse[:, None]) @ v
        got = batch.out[:, h * group:(h + 1) * group].double().reshape(-1, d)
        err = (got - ref).norm() / ref.norm()
        assert err <= (1e-5 if dtype == "f32" else 2e-3), (h, float(err))
        assert (batch.lse[:, h * group:(h + 1) * group].reshape(-1) - lse).abs().max() <= 2e-5
    B.ps_layout_release(pool, lay)
    B.ps_pool_destroy(pool)


@pytest.mark.parametrize("kv,q,d,heads", [("f32", "f32", 64, (4, 2)), ("f32", "f32", 256, (8, 4)), ("bf16", "bf16", 64, (16, 2)),
                                          ("bf16", "bf16", 256, (16, 4)), ("fp8_e4m3", "bf16", 64, (7, 1)), ("bf16", "f32", 128, (6, 2))])
def test_small_batches_in_items_of_16_rows(kv, q, d, heads):
    """Groups of up to 68 rows that a small batch sends out 16 rows at a time: a partly filled last item, and causal chunks whose rows
    see different lengths."""
    from paper_2602_12029_amd import binding as B
    geo = wl.Geometry(heads[0], heads[1], d, 16, q, kv)
    group = heads[0] // heads[1]
    new = 68 // group
    lens = [250 + new, 31 + new]
    w = wl.make_workload("narrow", geo, new, lens, [list(range(new))] * 2, [5, 33] + [0] * (2 * new - 2), pool_factor=1.3, seed=d)
    case = _case(w)
    for visible in (None, np.concatenate([np.arange(n - new, n) + 1 for n in lens]).astype(np.int32)):
        if visible is not None:
            case.set_visible(visible)
        items = B.ps_layout_plan(case.layout, w.num_requests)["items"]
        assert int(items[items[:, 7] & 1 == 0][:, 4].max()) * group <= 16
        _step(case, visible)
    case.close()
