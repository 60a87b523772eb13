"""GPU parity with per-request visible prefix lengths (partial prefill of new context tokens against the shared
cache): the HIP path through the C ABI against the fp64 oracle, element by element, same bars as the decode step."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase
    return GpuCase


def _run(case, visible, label, requests=None):
    from gpu_helpers import check_against_oracle
    case.poison_workspace()
    case.batch.decode_attention()
    return check_against_oracle(case, requests, label, visible, scaled_bar=True)   # rows that see a few tokens


def _variants(w):
    g = w.geometry
    return ["wave", "mfma"] if (g.q_dtype == "bf16" and g.kv_dtype != "f32" and g.head_dim == 128) else ["wave"]


def test_tiny_fp32_random_lengths(gpu):
    w = wl.named_workload("tiny")
    case = gpu(w)
    rng = np.random.default_rng(1)
    full = w.prefix_len[w.req_prompt]
    for trial, visible in enumerate([np.array([0, 256]), np.array([1, 255]), rng.integers(0, 257, 2), full]):
        for pc, sc in ((0, 0), (32, 32), (96, 4096)):
            case.replan(pc, sc)
            case.set_visible(visible)
            _run(case, visible, f"tiny visible {visible.tolist()} chunks {pc}/{sc}")
    case.set_visible(None)                                   # back to the plain decode step
    _run(case, None, "tiny, limits removed")
    case.close()


SHAPES = [
    ("vis_f32", wl.Geometry(4, 2, 64, 16, "f32", "f32"), 3, [1, 130, 517], [[0], [0, 2], [0, 1, 2]], [0, 33, 1, 16, 0, 250]),
    ("vis_bf16", wl.Geometry(32, 8, 128, 16, "bf16", "bf16"), 4, [700, 31, 1025], [[0, 1, 2, 3], [1], [0, 3]],
     [5, 0, 129, 64, 17, 1, 300]),
    ("vis_fp8", wl.Geometry(64, 8, 128, 16, "bf16", "fp8_e4m3"), 4, [515, 48], [[0, 1, 2, 3], [2, 3]],
     [1, 47, 0, 200, 16, 33]),
    ("vis_block64_fp8", wl.Geometry(16, 2, 128, 64, "bf16", "fp8_e4m3"), 3, [450, 64], [[0, 1, 2], [1]], [70, 1, 200, 129]),
    ("vis_many_rows", wl.Geometry(32, 2, 128, 16, "bf16", "bf16"), 10, [300], [list(range(10))], list(range(0, 10))),
]


@pytest.mark.parametrize("spec", SHAPES, ids=[s[0] for s in SHAPES])
def test_random_lengths_with_private_suffixes(gpu, spec):
    """Requests that see random parts of their prompt's prefix (none and all included) and keep their own suffix."""
    name, geo, models, prefix, membership, suffix = spec
    w = wl.make_workload(name, geo, models, prefix, membership, suffix, pool_factor=1.5, seed=29)
    case = gpu(w)
    rng = np.random.default_rng(31)
    full = w.prefix_len[w.req_prompt]
    for trial in range(3):
        visible = rng.integers(0, full + 1)
        visible[trial % len(visible)] = 0
        visible[(trial + 1) % len(visible)] = full[(trial + 1) % len(visible)]
        for variant in _variants(w):
            for pc, sc in ((0, 0), (64, 32), (256, 96)):
                case.replan(pc, sc, variant, variant)
                case.set_visible(visible)
                _run(case, visible, f"{name} #{trial} {variant} chunks {pc}/{sc}")
    case.close()


def test_nothing_visible_and_no_suffix_gives_zero_and_neg_inf(gpu):
    geo = wl.Geometry(8, 2, 128, 16, "bf16", "bf16")
    w = wl.make_workload("blind", geo, 3, [100], [[0, 1, 2]], [0, 0, 5], seed=37)
    case = gpu(w)
    visible = np.array([0, 60, 0])
    for variant in ("wave", "mfma"):
        case.replan(32, 32, variant, variant)
        case.set_visible(visible)
        _run(case, visible, f"blind {variant}")
        assert not case.batch.out[0].float().any() and torch.isneginf(case.batch.lse[0]).all()
    case.close()


CHUNKS = [
    # name, geometry, cached lengths, chunk lengths
    ("chunk_f32", wl.Geometry(4, 2, 64, 16, "f32", "f32"), [40, 7, 0], [19, 30, 5]),
    ("chunk_bf16", wl.Geometry(32, 8, 128, 16, "bf16", "bf16"), [1000, 0, 333], [200, 70, 17]),
    ("chunk_fp8", wl.Geometry(64, 8, 128, 16, "bf16", "fp8_e4m3"), [515, 2048], [100, 33]),
    ("chunk_block32_bf16", wl.Geometry(8, 2, 128, 32, "bf16", "bf16"), [300], [150]),
    # token ranges of one to four tiles, ending on, just before and just after a tile boundary, with 68 to 260 rows per
    # KV head: the first and last rounds of the prefill kernel's tile ring, waves without rows, partly filled row tiles
    ("chunk_edges_bf16", wl.Geometry(32, 8, 128, 16, "bf16", "bf16"), [0, 1, 31, 33, 64, 95], [17, 20, 33, 40, 64, 65]),
    ("chunk_edges_fp8_block32", wl.Geometry(64, 8, 128, 32, "bf16", "fp8_e4m3"), [0, 30, 63, 97], [9, 34, 33, 31]),
]


@pytest.mark.parametrize("spec", CHUNKS, ids=[s[0] for s in CHUNKS])
def test_causal_chunk_prefill(gpu, spec):
    """New context tokens prefilled against the cached context: token i of a chunk sees cached + i + 1 tokens."""
    name, geo, cached, chunk = spec
    w, visible = wl.chunk_prefill_workload(name, geo, cached, chunk, pool_factor=1.3, seed=41)
    case = gpu(w)
    for variant in _variants(w):
        for pc, sc in ((0, 0), (64, 32), (512, 96)):
            case.replan(pc, sc, variant, variant)
            case.set_visible(visible)
            _run(case, visible, f"{name} {variant} chunks {pc}/{sc}")
    case.close()


@pytest.mark.parametrize("name", ["prefill_b8", "prefill_fp8"])
def test_full_size_chunk_prefill_sampled_rows(gpu, name):
    """Benchmark-sized partial prefill, default plan: a seeded sample of query rows (first and last token of a
    chunk included) computed one by one by the oracle; every output finite; bitwise repeatable."""
    w, visible = wl.named_chunk_prefill(name)
    case = gpu(w)
    case.set_visible(visible)
    first_rows = np.flatnonzero(visible == visible.min())[:2].tolist()
    sample = sorted(set(np.random.default_rng(43).choice(w.num_requests, size=24, replace=False).tolist())
                    | set(first_rows) | {w.num_requests - 1})
    _run(case, visible, name, requests=sample)
    assert torch.isfinite(case.batch.out.float()).all()
    first = case.batch.out.clone()
    case.batch.decode_attention()
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), case.batch.out.view(torch.int16))
    case.close()


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
def test_rows_with_one_partial_state_match_the_merged_ones(gpu, kv_dtype):
    """The whole step stores the rows of requests with a single partial state from the prefill kernel; the two passes and
    the merge called one by one give the same bits -- whole contexts, cut ones, rows that see nothing, a context of few
    rows (the decode kernel), rows with a private suffix, with and without the log-sum-exp, and in place over q."""
    geo = wl.Geometry(32, 8, 128, 16, "bf16", kv_dtype)
    rng = np.random.default_rng(11)
    chunks, cached = [40, 7, 66, 33], [500, 90, 0, 2100]
    membership = [list(range(c)) for c in chunks]
    n = sum(chunks)
    suffix = np.where(np.arange(n) % 9 == 4, rng.integers(1, 40, n), 0)
    w = wl.make_workload("direct_" + kv_dtype, geo, max(chunks), [a + c for a, c in zip(cached, chunks)], membership,
                         suffix.tolist(), pool_factor=1.2, seed=29)
    visible = np.concatenate([a + 1 + np.arange(c) for a, c in zip(cached, chunks)]).astype(np.int32)
    visible[[3, 50, 100]] = 0
    case = gpu(w)
    for pc in (0, 256, 4096):
        case.replan(pc, 0)
        case.set_visible(visible)
        case.poison_workspace()
        case.batch.decode_attention()
        torch.cuda.synchronize()
        whole = case.batch.out.clone(), case.batch.lse.clone()
        case.poison_workspace()
        case.batch.prefix_attention()
        case.batch.suffix_attention()
        case.batch.merge_states()
        assert torch.equal(whole[0].view(torch.int16), case.batch.out.view(torch.int16))
        assert torch.equal(whole[1].view(torch.int32), case.batch.lse.view(torch.int32))
        case.poison_workspace()
        case.batch.decode_attention(with_lse=False)
        assert torch.equal(whole[0].view(torch.int16), case.batch.out.view(torch.int16))
        own_q, own_out = case.batch.q, case.batch.out
        case.batch.q = case.batch.out = own_q.clone()
        case.batch.decode_attention()
        assert torch.equal(whole[0].view(torch.int16), case.batch.out.view(torch.int16))
        case.batch.q, case.batch.out = own_q, own_out
    case.close()


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
def test_the_whole_step_leaves_every_partial_state(gpu, kv_dtype):
    """The workspace holds the same states after the whole step as after its two passes, rows that are stored without a merge
    included, so that a merge behind it gives the same output; the step on the library's own buffer gives it too."""
    from paper_2602_12029_amd import binding as B
    geo = wl.Geometry(32, 8, 128, 16, "bf16", kv_dtype)
    w, visible = wl.chunk_prefill_workload("states_" + kv_dtype, geo, [500, 90, 2100, 20], [40, 66, 33, 3], pool_factor=1.2, seed=37)
    case = gpu(w)
    for pc in (0, 512, 4096):
        case.replan(pc, 0)
        case.set_visible(visible)
        case.poison_workspace()
        case.batch.prefix_attention()
        case.batch.suffix_attention()
        want = case.batch.workspace.clone()
        case.poison_workspace()
        case.batch.decode_attention()
        assert torch.equal(case.batch.workspace, want)
        out, lse = case.batch.out.clone(), case.batch.lse.clone()
        case.batch.out.zero_()
        case.batch.merge_states()
        assert torch.equal(out.view(torch.int16), case.batch.out.view(torch.int16))
        assert torch.equal(lse.view(torch.int32), case.batch.lse.view(torch.int32))
        case.poison_workspace()
        b = case.batch
        B.ps_decode_attention_static(case.layout, b.tables.data_ptr(), b.q.data_ptr(), b.kv.data_ptr(),
                                     b.scales.data_ptr() if b.scales is not None else 0, b.out.data_ptr(), b.lse.data_ptr(),
                                     torch.cuda.current_stream().cuda_stream)
        assert torch.equal(out.view(torch.int16), b.out.view(torch.int16)) and torch.equal(lse.view(torch.int32), b.lse.view(torch.int32))
        own = b.out                                      # an output off a 16-byte boundary
        b.out = torch.zeros(own.numel() + 8, dtype=own.dtype, device="cuda")[4:4 + own.numel()].view(own.shape)
        assert b.out.data_ptr() % 16 == 8
        b.decode_attention()
        assert torch.equal(out.view(torch.int16), b.out.view(torch.int16))
        b.out = own
    case.close()


@pytest.mark.parametrize("heads,rows", [((32, 8), 128), ((64, 8), 256)])
@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
def test_prefill_ring_edges(gpu, kv_dtype, heads, rows):
    """Token ranges that end in and around each of the first ten tiles: a ring of three stages of one or two tiles, filled
    up to six tiles ahead, by four and by eight waves; waves with all, some and none of their rows."""
    from paper_2602_12029_amd import binding as B
    geo = wl.Geometry(heads[0], heads[1], 128, 16, "bf16", kv_dtype)
    cached = [32 * k + e for k in range(0, 10) for e in (-20, -19, -18)][3:]
    chunk = [18 + (i % 3) * 7 for i in range(len(cached))]
    w, visible = wl.chunk_prefill_workload("ring_" + kv_dtype, geo, cached, chunk, pool_factor=1.2, seed=31)
    case = gpu(w)
    case.set_visible(visible)
    items = B.ps_layout_plan(case.layout, w.num_requests)["items"]
    most = int(items[(items[:, 7] & 4) != 0][:, 4].max()) * geo.group
    assert (most <= 128) if rows == 128 else (128 < most <= 256)
    _run(case, visible, w.name)
    case.close()


@pytest.mark.parametrize("heads,rows", [((32, 8), 128), ((64, 8), 256)])
@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
def test_prefill_tiles_past_the_range_in_large_blocks(gpu, kv_dtype, heads, rows):
    """A tile past an item's tokens repeats the range's last 16-token block: ranges that end in each quarter of a block of 64,
    whose slots behind them are poisoned, at every remainder of the four tiles the eight-wave loop takes at a time."""
    from paper_2602_12029_amd import binding as B
    geo = wl.Geometry(heads[0], heads[1], 128, 64, "bf16", kv_dtype)
    cached = [16 * k + 1 for k in range(4, 22)]
    chunk = [24 + (i % 3) * 7 for i in range(len(cached))]
    w, visible = wl.chunk_prefill_workload("past_" + kv_dtype, geo, cached, chunk, pool_factor=1.2, seed=33)
    case = gpu(w)
    case.set_visible(visible)
    items = B.ps_layout_plan(case.layout, w.num_requests)["items"]
    most = int(items[(items[:, 7] & 4) != 0][:, 4].max()) * geo.group
    assert (most <= 128) if rows == 128 else (128 < most <= 256)
    _run(case, visible, w.name)
    case.close()
