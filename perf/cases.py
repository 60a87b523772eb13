"""Timed cases: the work a serving program has this library do, through its public entry points.

A case names a path and the sizes of a batch:

  decode   one decode-attention step over a batch that is already laid out
  step     the device side of one decode step: the step's new K/V rows stored, then the attention
  prefill  partial prefill: attention of the tokens newly appended to cached contexts
  ingest   hand-off of a batch's K/V (shared prefixes, private suffixes) into the paged pool
  stage    the batch's blocks out to a staging image in device memory and back
  turn     one agent turn: a batch laid out over cached contexts, a few decode steps with cache growth, release

Lengths follow from the case alone (its `lens` seed), values and block placement from the seed given to prepare().
Queries and keys are N(0,1) with a sink: the first four tokens of a shared segment score a few units above the rest, as
attention sinks do.
"""
import math

import numpy as np
import torch

from paper_2602_12029_amd import binding as B
from paper_2602_12029_amd.runtime import DecodeBatch

ESZ = {"f32": 4, "bf16": 2, "fp8_e4m3": 1}
SINK_TOKENS, SINK_Q, SINK_K = 4, 0.5, 1.0


def _case(path, kv, heads, prompts, models, prefix, suffix, block=16, root=0, spread="uniform", steps=0, lens=0, **more):
    return dict(path=path, kv=kv, q_heads=heads[0], kv_heads=heads[1], head_dim=heads[2], block=block, prompts=prompts,
                models_lo=models[0], models_hi=models[1], prefix_lo=prefix[0], prefix_hi=prefix[1], spread=spread,
                suffix_lo=suffix[0], suffix_hi=suffix[1], root=root, steps=steps, lens=lens, **more)


H8B, H70B, H64 = (32, 8, 128), (64, 8, 128), (32, 8, 64)


def listed():
    return [
        # the smallest batch of the benchmark configurations: two models on one short prompt, fp32 (launch latency)
        _case("decode", "f32", (4, 2, 64), 1, (2, 2), (256, 256), (8, 8), name="tiny_f32"),
        # a lone agent session, four decode models on one context: what an otherwise idle GPU answers with
        _case("step", "bf16", H8B, 1, (4, 4), (2741, 2741), (1, 256), lens=1, name="one_session"),
        # a moderately loaded decode GPU: forty four-agent sessions with contexts of ragged lengths
        _case("step", "bf16", H8B, 40, (4, 4), (1024, 6144), (1, 256), lens=2, name="sessions40"),
        # the largest benchmark configuration: 256 prompts, log-uniform contexts, 2 to 6 models on each
        _case("decode", "bf16", H8B, 256, (2, 6), (512, 16384), (1, 1024), spread="log", lens=3, name="mixed"),
        # a 70B-shaped model with e4m3 KV under four models
        _case("decode", "fp8_e4m3", H70B, 64, (4, 4), (8192, 8192), (1, 512), lens=4, name="fp8_70b"),
        # float32 caches, as used where outputs are compared against a reference or a model runs in full precision
        _case("decode", "f32", H8B, 12, (2, 4), (512, 4096), (1, 256), lens=5, name="f32_sessions"),
        # a small model with 64-wide heads, blocks of 32 tokens
        _case("decode", "bf16", H64, 24, (2, 4), (1024, 6144), (1, 256), block=32, lens=6, name="d64_sessions"),
        # segments handed from one agent to the next: 32 contexts grow by up to 256 tokens each
        _case("prefill", "bf16", H8B, 32, (1, 1), (4096, 4096), (64, 256), lens=7, name="prefill_b8"),
        # the same with a 70B-shaped model, e4m3 KV and longer contexts
        _case("prefill", "fp8_e4m3", H70B, 64, (1, 1), (8192, 8192), (64, 256), lens=8, name="prefill_fp8"),
        # a prefill worker's K/V handed over and quantised to e4m3
        _case("ingest", "fp8_e4m3", H70B, 48, (4, 4), (2048, 12288), (1, 512), lens=9, name="ingest_fp8"),
        # a batch of cold sessions staged out and back in
        _case("stage", "bf16", H8B, 32, (4, 4), (1024, 6144), (1, 512), lens=10, name="stage_b8"),
        # one agent turn over sixteen cached contexts: four models decode eight tokens each
        _case("turn", "bf16", H8B, 16, (4, 4), (1024, 6144), (0, 0), steps=8, lens=11, name="turn16"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    path = rng.choice(["decode", "decode", "decode", "step", "prefill", "prefill", "ingest", "stage", "turn"])
    kind = rng.choice(["bf16", "bf16", "fp8_e4m3", "f32", "narrow", "wide"])
    if path in ("ingest", "stage", "turn") and kind in ("narrow", "wide"):
        kind = "bf16"
    kv = {"narrow": "bf16", "wide": "bf16"}.get(kind, kind)
    heads = {"bf16": rng.choice([H8B, H8B, (64, 8, 128), (16, 8, 128), (28, 4, 128)]),
             "fp8_e4m3": rng.choice([H70B, H8B]),
             "f32": rng.choice([H8B, (4, 2, 64), (16, 8, 128), (8, 4, 256)]),
             "narrow": rng.choice([H64, (16, 2, 64)]), "wide": (16, 4, 256)}[kind]
    block = rng.choice([16, 16, 16, 32, 64])
    token = 2 * heads[1] * heads[2] * ESZ[kv]              # bytes of K and V of one token
    general = kind in ("f32", "narrow", "wide")
    if path == "prefill":
        # flops: 4 d per q head and visible token
        prompts, cached = log_int(1, 4 if general else 48), log_int(64, 2048 if general else 12000)
        chunk = rng.randint(8, 48 if general else 256)
        most = 1.5e10 if general else 1.8e12
        while prompts > 1 and 4.0 * heads[2] * heads[0] * prompts * chunk * cached > most:
            prompts -= 1
        return _case(path, kv, heads, prompts, (1, 1), (max(1, cached // 2), cached), (max(1, chunk // 4), chunk),
                     block=block, lens=rng.randrange(1 << 20))
    prompts, longest = log_int(1, 192), log_int(96, 24000)
    models = rng.randint(1, 8)
    suffix = log_int(4, 1024)
    most = {"decode": 5.0e9, "step": 5.0e9, "ingest": 1.2e9, "stage": 1.0e9, "turn": 4.0e8}[path]
    if general:
        most = min(most, 6.0e8)
    while prompts > 1 and prompts * (longest + models * suffix / 2.0) * token > most:
        prompts = prompts * 3 // 4
    while (longest + models * suffix / 2.0) * token > most:
        longest, suffix = longest * 3 // 4, max(4, suffix * 3 // 4)
    root = log_int(32, 4096) if path == "decode" and prompts > 1 and rng.random() < 0.25 else 0
    return _case(path, kv, heads, prompts, (rng.randint(1, models), models), (max(1, longest // rng.choice([1, 4, 16])), longest),
                 (0, 0) if path == "turn" else (1, suffix), block=block, root=root, spread=rng.choice(["uniform", "log"]),
                 steps=rng.randint(2, 12) if path == "turn" else 0, lens=rng.randrange(1 << 20))


# ---- lengths and tables --------------------------------------------------------------------------------------

class Lengths:
    """Segment lengths and requests of a case (prompt-major), from its own seed."""

    def __init__(self, case):
        rng = np.random.default_rng([17, case["lens"]])
        n, lo, hi = case["prompts"], case["prefix_lo"], case["prefix_hi"]
        if case["spread"] == "log" and hi > lo:
            prefix = np.clip(np.floor(np.exp(rng.uniform(math.log(lo), math.log(hi + 1), n))), lo, hi).astype(np.int32)
        else:
            prefix = rng.integers(lo, hi + 1, n).astype(np.int32)
        self.cached = prefix
        self.visible = None
        if case["path"] == "prefill":       # every new token is a request that sees the context up to itself
            chunk = rng.integers(case["suffix_lo"], case["suffix_hi"] + 1, n).astype(np.int32)
            counts = chunk
            prefix = prefix + chunk
        else:
            counts = rng.integers(case["models_lo"], case["models_hi"] + 1, n)
        self.prefix = prefix.astype(np.int32)
        self.req_prompt = np.repeat(np.arange(n, dtype=np.int32), counts)
        self.req_model = np.concatenate([np.arange(c, dtype=np.int32) for c in counts])
        self.num_requests = int(self.req_prompt.size)
        if case["path"] == "prefill":
            self.visible = (self.cached[self.req_prompt] + self.req_model + 1).astype(np.int32)
            self.suffix = np.zeros(self.num_requests, np.int32)
        else:
            self.suffix = rng.integers(case["suffix_lo"], case["suffix_hi"] + 1, self.num_requests).astype(np.int32)
        self.root = np.array([case["root"]] if case["root"] else [], np.int32)
        # half of the prompts begin with the root, where there is one
        self.prompt_root = np.where(np.arange(n) % 2 == 0, 0, -1).astype(np.int32) if case["root"] else None

    def blocks(self, block, extra_tokens=0):
        up = lambda x: int(((x.astype(np.int64) + block - 1) // block).sum())   # noqa: E731
        return up(self.prefix) + up(self.root) + up(self.suffix + extra_tokens)


def _tables(case, lens, order):
    """Block ids of every segment by the documented policy: roots, prompts, requests take theirs from the head of the
    free list; the token a step appends takes one more block where the private segment is at a block boundary."""
    at, out = 0, {"root": [], "prefix": [], "suffix": []}
    for kind, seg in (("root", lens.root), ("prefix", lens.prefix), ("suffix", lens.suffix)):
        for length in seg:
            n = -(-int(length) // case["block"])
            out[kind].append(order[at:at + n])
            at += n
    if case["path"] == "step":
        for r, length in enumerate(lens.suffix):
            if length % case["block"] == 0:
                out["suffix"][r] = np.append(out["suffix"][r], order[at])
                at += 1
    return out


# ---- inputs ---------------------------------------------------------------------------------------------------

def _dtype(kv):
    return torch.float32 if kv == "f32" else torch.bfloat16


def _direction(case, device="cuda"):
    """A fixed sign pattern over the head dimension: queries lean along it, and so do the sink tokens' keys."""
    return torch.from_numpy(np.random.default_rng(3).choice([-1.0, 1.0], case["head_dim"]).astype(np.float32)).to(device)


def _inputs(case, seed):
    """Pool contents, queries and block order of one seed (nothing here depends on this repository's code)."""
    lens = Lengths(case)
    gen = torch.Generator(device="cuda").manual_seed(1000003 * (seed % (1 << 32)) + 7)
    h, d, blk, kv = case["kv_heads"], case["head_dim"], case["block"], case["kv"]
    spare = case["steps"] + (1 if case["path"] == "step" else 0)
    num_blocks = lens.blocks(blk, spare) + 3
    if case["path"] == "turn":
        num_blocks += case["prompts"]                  # a turn takes a block of its own for the tail of each context
    order = np.random.default_rng([seed, 5]).permutation(num_blocks).astype(np.int32)
    shape = (num_blocks, h, 2, blk, d)
    u = _direction(case)
    tables = _tables(case, lens, order)
    pool = torch.empty(shape, dtype=torch.uint8 if kv == "fp8_e4m3" else _dtype(kv), device="cuda")
    scales = None
    if kv == "fp8_e4m3":
        scales = (0.95 + 0.1 * torch.rand((num_blocks, h, 2), device="cuda", generator=gen)) / 100.0
    firsts = [ids[0] for ids in tables["root"] + tables["prefix"] if len(ids)]
    firsts = torch.from_numpy(np.array(firsts, np.int64)).cuda()
    sink = torch.zeros((2, blk, d), device="cuda")
    sink[0, :min(SINK_TOKENS, blk)] = SINK_K * u
    if case["path"] != "ingest":
        per = max(1, (1 << 27) // (h * 2 * blk * d))
        for b0 in range(0, num_blocks, per):
            x = torch.randn((min(per, num_blocks - b0), h, 2, blk, d), device="cuda", generator=gen)
            mine = firsts[(firsts >= b0) & (firsts < b0 + per)] - b0
            x[mine] += sink
            if kv == "fp8_e4m3":
                code = (x / scales[b0:b0 + per, :, :, None, None]).clamp_(-448, 448).to(torch.float8_e4m3fn)
                pool[b0:b0 + per] = code.view(torch.uint8)
            else:
                pool[b0:b0 + per] = x.to(pool.dtype)
    else:
        pool.zero_()
        if scales is not None:
            scales.zero_()

    def queries():
        x = torch.randn((lens.num_requests, case["q_heads"], d), device="cuda", generator=gen) + SINK_Q * u
        return x.to(_dtype(kv))

    def rows(tokens):
        x = torch.randn((tokens, h, d), device="cuda", generator=gen)
        gain = torch.exp2(-2.0 * torch.rand((tokens, 1, 1), device="cuda", generator=gen))
        return (x * gain).to(_dtype(kv))

    got = {"lens": lens, "order": order, "num_blocks": num_blocks, "pool": pool, "scales": scales, "tables": tables}
    if case["path"] in ("decode", "step", "prefill"):
        got["q"] = queries()
    if case["path"] == "step":
        got["new"] = (rows(lens.num_requests), rows(lens.num_requests))
    if case["path"] == "ingest":
        got["src"] = [(rows(int(n)), rows(int(n))) for n in (lens.prefix.sum(dtype=np.int64), lens.suffix.sum(dtype=np.int64))]
    if case["path"] == "turn":
        got["q"] = [queries() for _ in range(case["steps"])]
        got["new"] = [(rows(lens.num_requests), rows(lens.num_requests)) for _ in range(case["steps"])]
        tail = int((lens.prefix % blk).sum())          # tokens past the last full block of each context
        got["tail"] = (rows(tail), rows(tail))
    return got


def prepare(case, seed):
    s = _inputs(case, seed)
    lens, path = s["lens"], case["path"]
    q_dtype = "f32" if case["kv"] == "f32" else "bf16"
    geo = B.geometry(case["q_heads"], case["kv_heads"], case["head_dim"], case["block"], q_dtype, case["kv"])
    pool = B.ps_pool_create(s["num_blocks"], s["order"])
    state = {"case": case, "geo": geo, "pool": pool, "kv": s["pool"], "scales": s["scales"]}
    if path == "turn":
        # the contexts are cached: a layout holds their blocks, a turn adopts the full ones
        one = np.arange(case["prompts"], dtype=np.int32)
        keep = B.ps_kv_layout(pool, geo, lens.prefix, one, np.zeros_like(one), np.zeros_like(one))
        t = B.ps_layout_tables(keep, case["prompts"], case["prompts"])
        ip = t["prefix_blk_indptr"]
        adopt = [t["prefix_blk"][ip[p]:ip[p] + lens.prefix[p] // case["block"]] for p in range(case["prompts"])]
        state.update(keep=keep, adopt=adopt, lens=lens, q=s["q"], new=s["new"], tail=s["tail"])
        return state
    if lens.root.size:
        layout = B.ps_kv_layout_tree(pool, geo, lens.root, lens.prompt_root, lens.prefix, lens.req_prompt, lens.req_model,
                                     lens.suffix)
    else:
        layout = B.ps_kv_layout(pool, geo, lens.prefix, lens.req_prompt, lens.req_model, lens.suffix)
    if path == "step":                                   # the host side of the step: where its tokens go
        B.ps_layout_append(pool, layout, lens.num_requests)
        state["new"] = s["new"]
    q = s.get("q")
    if q is None:
        q = torch.zeros((lens.num_requests, case["q_heads"], case["head_dim"]), dtype=_dtype(case["kv"]), device="cuda")
    state["layout"] = layout
    state["batch"] = batch = DecodeBatch(layout, geo, lens.num_requests, q, s["pool"], s["scales"])
    if path == "prefill":
        batch.set_visible(lens.visible)
    if path == "ingest":
        state["src"] = s["src"]
    if path == "stage":
        state["image"] = torch.zeros(B.ps_stage_layout(layout)[2], dtype=torch.uint8, device="cuda")
    return state


# ---- one pass ---------------------------------------------------------------------------------------------------

def _stream():
    return int(torch.cuda.current_stream().cuda_stream)


def _cache(state):
    return {"kv": state["kv"]} if state["scales"] is None else {"kv": state["kv"], "scales": state["scales"]}


def run(state):
    path = state["case"]["path"]
    if path == "turn":
        return _turn(state)
    batch = state["batch"]
    if path == "ingest":
        for which, (k, v) in enumerate(state["src"]):
            batch.kv_ingest(which, k, v)
        return _cache(state)
    if path == "stage":
        batch.stage_out(state["image"])
        batch.stage_in(state["image"])
        return {"image": state["image"], **_cache(state)}
    if path == "step":
        new_k, new_v = state["new"]
        B.ps_kv_append(state["layout"], batch.tables.data_ptr(), new_k.data_ptr(), new_v.data_ptr(), batch.kv.data_ptr(),
                       batch.scales.data_ptr() if batch.scales is not None else 0, _stream())
        batch.decode_attention()
        return {"out": batch.out, "lse": batch.lse, **_cache(state)}
    batch.decode_attention()
    return {"out": batch.out, "lse": batch.lse}


def _turn(state):
    lens = state["lens"]
    layout = B.ps_kv_layout_adopt(state["pool"], state["geo"], lens.prefix, state["adopt"], lens.req_prompt, lens.req_model,
                                  lens.suffix)
    batch = DecodeBatch(layout, state["geo"], lens.num_requests, state["q"][0], state["kv"], state["scales"])
    batch.kv_ingest(0, *state["tail"])
    outs = []
    for q, (new_k, new_v) in zip(state["q"], state["new"]):
        batch.append_step(state["pool"], new_k, new_v)
        batch.q = q
        batch.decode_attention()
        outs.append(batch.out.clone())
    B.ps_layout_release(state["pool"], layout)
    return {"out": outs, "lse": batch.lse}


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def work(case):
    lens = Lengths(case)
    hq, h, d, blk, esz = case["q_heads"], case["kv_heads"], case["head_dim"], case["block"], ESZ[case["kv"]]
    qsz = 4 if case["kv"] == "f32" else 2
    token = 2 * h * d * esz
    tile_scales = 8 * h if case["kv"] == "fp8_e4m3" else 0
    shared = int(lens.prefix.sum(dtype=np.int64) + lens.root.sum(dtype=np.int64))
    own = int(lens.suffix.sum(dtype=np.int64))
    n = lens.num_requests
    rows = n * hq * (2 * d * qsz + 4)                   # queries in, outputs and log-sum-exps out
    seen = lens.visible.astype(np.int64) if lens.visible is not None else lens.prefix.astype(np.int64)[lens.req_prompt]
    if lens.root.size:
        seen = seen + np.where(lens.prompt_root[lens.req_prompt] == 0, int(lens.root[0]), 0)
    blocks = lens.blocks(blk)
    if case["path"] == "ingest":
        tokens = shared + own
        return {"bytes": tokens * 2 * h * d * qsz + tokens * token + blocks * tile_scales, "flops": 0}
    if case["path"] == "stage":
        return {"bytes": 4 * blocks * (blk * token + tile_scales), "flops": 0}
    flops = 4 * d * hq * int((seen + lens.suffix).sum())
    total = (shared + own) * token + blocks * tile_scales + rows
    if case["path"] == "step":
        total += n * (2 * h * d * qsz + token)
        flops += 4 * d * hq * n
    if case["path"] == "turn":
        steps = case["steps"]
        tail = int((lens.prefix % blk).sum())
        grown = n * steps * (steps + 1) // 2
        total = steps * (shared * token + blocks * tile_scales + rows) + grown * token + (steps * n + tail) * (2 * h * d * qsz + token)
        flops = 4 * d * hq * (steps * int(seen.sum()) + grown)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["path"] in ("ingest", "stage"):
        return "exact"                                  # bytes are copied, codes are defined bit by bit
    if case["kv"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    # bf16 outputs, probabilities in 16 bits on the matrix cores
    return {"rel": 1e-2, "max": 0.1}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------

def _segment(case, s, ids, length):
    """K, V of a segment as [heads, length, d] in 64 bits, from the pool."""
    idx = torch.from_numpy(np.asarray(ids, np.int64)).cuda()
    x = s["pool"][idx]
    if case["kv"] == "fp8_e4m3":
        x = x.view(torch.float8_e4m3fn).to(torch.float32).to(torch.float64) * s["scales"][idx].to(torch.float64)[:, :, :, None, None]
    x = x.to(torch.float64).permute(2, 1, 0, 3, 4).reshape(2, case["kv_heads"], -1, case["head_dim"])[:, :, :length]
    return x[0].contiguous(), x[1].contiguous()


def _attend(case, s, q_all, suffix_of, prefix_of, out, lse):
    """Fills out [R, Hq, d], lse [R, Hq]: softmax attention of every request over [root ; prefix ; suffix]."""
    lens = s["lens"]
    h, g, d = case["kv_heads"], case["q_heads"] // case["kv_heads"], case["head_dim"]
    scale = 1.0 / math.sqrt(d)
    for p in range(case["prompts"]):
        reqs = np.nonzero(lens.req_prompt == p)[0]
        k, v = prefix_of(p)
        if lens.root.size and lens.prompt_root[p] == 0:
            rk, rv = _segment(case, s, s["tables"]["root"][0], int(lens.root[0]))
            k, v = torch.cat([rk, k], 1), torch.cat([rv, v], 1)
        at = torch.from_numpy(reqs).cuda()
        q = q_all[at].to(torch.float64).reshape(len(reqs), h, g, d)
        if lens.visible is not None:
            see = torch.from_numpy(lens.visible[reqs]).cuda()
            hidden = torch.arange(k.shape[1], device="cuda")[None, :] >= see[:, None]
            hidden = hidden.repeat_interleave(g, 0)
            for i in range(h):
                sc = (q[:, i].reshape(-1, d) @ k[i].t().contiguous()) * scale
                sc.masked_fill_(hidden, -math.inf)
                top = torch.logsumexp(sc, 1)
                lse[at, i * g:(i + 1) * g] = top.reshape(-1, g)
                out[at, i * g:(i + 1) * g] = (torch.exp(sc - top[:, None]) @ v[i]).reshape(-1, g, d)
            continue
        kt = k.transpose(1, 2).contiguous()
        rows = q.permute(1, 0, 2, 3).reshape(h, -1, d).contiguous()
        shared = (torch.bmm(rows, kt) * scale).reshape(h, len(reqs), g, -1)
        for j, r in enumerate(reqs.tolist()):
            sk, sv = suffix_of(r)
            own = torch.bmm(q[j], sk.transpose(1, 2).contiguous()) * scale
            sc = torch.cat([shared[:, j], own], 2)
            top = torch.logsumexp(sc, 2)
            w = torch.exp(sc - top[:, :, None])
            n = shared.shape[3]
            lse[r] = top.reshape(-1)
            out[r] = (torch.bmm(w[:, :, :n].contiguous(), v) + torch.bmm(w[:, :, n:].contiguous(), sv)).reshape(-1, d)


def exact(case, seed):
    path = case["path"]
    if path in ("ingest", "stage") or (path in ("step", "turn") and case["kv"] == "fp8_e4m3"):
        return None                                     # bytes; or values that went through the e4m3 quantiser
    s = _inputs(case, seed)
    lens, t = s["lens"], s["tables"]
    shape = (lens.num_requests, case["q_heads"], case["head_dim"])

    def fresh():
        return (torch.zeros(shape, dtype=torch.float64, device="cuda"),
                torch.zeros(shape[:2], dtype=torch.float64, device="cuda"))

    def prefix_of(p):
        k, v = _segment(case, s, t["prefix"][p], int(lens.prefix[p]))
        if path == "turn":
            n = int(lens.prefix[p] % case["block"])
            if n:
                first = int((lens.prefix[:p] % case["block"]).sum())
                for x, src in ((k, s["tail"][0]), (v, s["tail"][1])):
                    x[:, x.shape[1] - n:] = src[first:first + n].to(torch.float64).transpose(0, 1)
        return k, v

    if path == "turn":
        outs = []
        for i in range(case["steps"]):
            new_k = torch.stack([k for k, _ in s["new"][:i + 1]], 1).to(torch.float64)      # [R, tokens, heads, d]
            new_v = torch.stack([v for _, v in s["new"][:i + 1]], 1).to(torch.float64)
            out, lse = fresh()
            _attend(case, s, s["q"][i], lambda r: (new_k[r].transpose(0, 1).contiguous(), new_v[r].transpose(0, 1).contiguous()),
                    prefix_of, out, lse)
            outs.append(out)
        return {"out": outs, "lse": lse}

    def suffix_of(r):
        n = int(lens.suffix[r])
        k, v = _segment(case, s, t["suffix"][r], n + (1 if path == "step" else 0))
        if path == "step":
            k[:, n], v[:, n] = s["new"][0][r].to(torch.float64), s["new"][1][r].to(torch.float64)
        return k, v

    out, lse = fresh()
    _attend(case, s, s["q"], suffix_of, prefix_of, out, lse)
    if path == "step":
        return {"out": out, "lse": lse, "kv": None}
    return {"out": out, "lse": lse}
