"""GPU: ps_merge_states on caller-built partial states, at the edges of its rounds (4 and 16 states per round trip).

Bars: float32 outputs 1e-5 absolute (a weighted mean of a few dozen N(0,1) values); bf16 outputs one rounding, 2^-8 of the
largest output."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import attention as oa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("states", [[1, 4, 2, 3], [5, 1, 16, 4], [15, 17, 2, 1], [33, 16, 32, 0]])
def test_rounds_of_the_merge(states, q_dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase
    from paper_2602_12029_amd import binding as B
    geo = wl.Geometry(4, 2, 64, 16, q_dtype, q_dtype)
    w = wl.make_workload("merge", geo, 2, [32 * n for n in states], [[0, 1]] * len(states), [0] * (2 * len(states)), seed=5)
    case = GpuCase(w)
    case.replan(32, 32)
    o_ws, lse_ws = case.batch.workspace_views()
    gen = torch.Generator().manual_seed(7)
    o = torch.randn(o_ws.shape, generator=gen)
    lse = torch.randn(lse_ws.shape, generator=gen) * 3
    lse[::7] = float("-inf")          # empty partial states
    o[::7] = float("nan")             # ... whose values count for nothing
    o_ws.copy_(o)
    lse_ws.copy_(lse)
    case.batch.merge_states()
    torch.cuda.synchronize()
    base = B.ps_layout_plan(case.layout, w.num_requests)["slot_base"]
    assert [int(base[2 * p + 1] - base[2 * p]) for p in range(len(states))] == states
    got, got_lse = case.batch.out.float().cpu().double().numpy(), case.batch.lse.cpu().double().numpy()
    for r in range(w.num_requests):
        s = slice(base[r], base[r + 1])
        ro, rl = oa.merge_states(torch.nan_to_num(o[s]).double().numpy(), lse[s].double().numpy())
        if states[r // 2] == 0:
            ro, rl = np.zeros((4, 64)), np.full(4, -np.inf)
        bar = 1e-5 if q_dtype == "f32" else max(1e-5, np.abs(ro).max() * 2.0 ** -8)
        assert np.abs(got[r] - ro).max() <= bar
        assert np.array_equal(np.isneginf(got_lse[r]), np.isneginf(rl))
        some = np.isfinite(rl)
        assert np.abs(got_lse[r][some] - rl[some]).max(initial=0.0) <= 1e-5
    case.close()


@pytest.mark.parametrize("q_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,heads,states", [
    (64, 4, [5, 17, 64, 65, 0]), (128, 4, [8, 9, 31, 33, 100]), (256, 4, [4, 5, 16, 17, 40]),   # a workgroup per row, around its rounds
    (128, 64, [5, 16, 7, 1, 12]), (64, 256, [17, 33, 2, 16, 5])])                                # more rows: a thread per four columns
def test_rows_of_many_states(d, heads, states, q_dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase
    from paper_2602_12029_amd import binding as B
    geo = wl.Geometry(heads, 2, d, 16, q_dtype, q_dtype)
    w = wl.make_workload("many", geo, 2, [32 * n for n in states], [[0, 1]] * len(states), [0] * (2 * len(states)), seed=6)
    case = GpuCase(w)
    case.replan(32, 32, "wave", "wave")
    o_ws, lse_ws = case.batch.workspace_views()
    gen = torch.Generator().manual_seed(d + heads)
    o = torch.randn(o_ws.shape, generator=gen)
    lse = torch.randn(lse_ws.shape, generator=gen) * 3
    lse[::5] = float("-inf")          # empty partial states
    o[::5] = float("nan")             # ... whose values count for nothing
    o_ws.copy_(o)
    lse_ws.copy_(lse)
    case.batch.merge_states()
    torch.cuda.synchronize()
    base = B.ps_layout_plan(case.layout, w.num_requests)["slot_base"]
    assert [int(base[2 * p + 1] - base[2 * p]) for p in range(len(states))] == states
    got, got_lse = case.batch.out.float().cpu().double().numpy(), case.batch.lse.cpu().double().numpy()
    for r in range(w.num_requests):
        s = slice(base[r], base[r + 1])
        ro, rl = oa.merge_states(torch.nan_to_num(o[s]).double().numpy(), lse[s].double().numpy())
        if states[r // 2] == 0:
            ro, rl = np.zeros((heads, d)), np.full(heads, -np.inf)
        bar = 1e-5 if q_dtype == "f32" else max(1e-5, np.abs(ro).max() * 2.0 ** -8)
        assert np.abs(got[r] - ro).max() <= bar
        assert np.array_equal(np.isneginf(got_lse[r]), np.isneginf(rl))
        some = np.isfinite(rl)
        assert np.abs(got_lse[r][some] - rl[some]).max(initial=0.0) <= 1e-5
    case.close()


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("heads,states", [(4, [8, 5, 33, 1, 3]), (128, [8, 5, 16, 1, 3]), (256, [17, 33, 2, 16, 4])])   # a workgroup per row; a thread per four columns
def test_a_state_that_is_not_a_number(d, heads, states):
    """A log-sum-exp that is not a number makes its row not a number, whichever states stand beside it: finite ones, empty ones, none;
    the other heads of the request keep their values."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_helpers import GpuCase
    from paper_2602_12029_amd import binding as B
    geo = wl.Geometry(heads, 2, d, 16, "f32", "f32")
    w = wl.make_workload("nan", geo, 2, [32 * n for n in states], [[0, 1]] * len(states), [0] * (2 * len(states)), seed=8)
    case = GpuCase(w)
    case.replan(32, 32, "wave", "wave")
    o_ws, lse_ws = case.batch.workspace_views()
    gen = torch.Generator().manual_seed(d + heads)
    o = torch.randn(o_ws.shape, generator=gen)
    lse = torch.randn(lse_ws.shape, generator=gen) * 3
    base = B.ps_layout_plan(case.layout, w.num_requests)["slot_base"]
    for r in range(w.num_requests):
        n = int(base[r + 1] - base[r])
        lse[int(base[r]) + n // 2, 0] = float("nan")       # one of several
        lse[int(base[r]):int(base[r + 1]), 1] = float("nan")   # all
        lse[int(base[r]):int(base[r + 1]), 2] = float("-inf")  # the only one that is not empty
        lse[int(base[r]) + n - 1, 2] = float("nan")
    o_ws.copy_(o)
    lse_ws.copy_(lse)
    case.batch.merge_states()
    torch.cuda.synchronize()
    got, got_lse = case.batch.out.cpu(), case.batch.lse.cpu()
    assert torch.isnan(got[:, :3]).all() and torch.isnan(got_lse[:, :3]).all()
    for r in range(w.num_requests):
        s = slice(base[r], base[r + 1])
        ro, rl = oa.merge_states(o[s, 3:].double().numpy(), lse[s, 3:].double().numpy())
        assert np.abs(got[r, 3:].double().numpy() - ro).max() <= 1e-5
        assert np.abs(got_lse[r, 3:].double().numpy() - rl).max() <= 1e-5
    case.close()
