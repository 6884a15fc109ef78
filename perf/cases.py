"""Performance cases: what a user of this framework has it do, over the sizes it is used at.

The sizes are those of the workload configurations (paper_2507_00715_amd/workloads.py) and of the benchmark's further
figures: the whole path of a request batch, one full-length prefill layer, one decode step of a whole model, one
beam-search step, the dense products of a decoder layer, and the attention of a training step.  Inputs are drawn from
N(0, 1) like the workloads' own (scaled weights, occasional large keys where a configuration has them); sequence lengths
are part of a case (`lengths_seed`), so a case is the same amount of work whatever the inputs' seed.
"""
import math
import random

import torch

from paper_2507_00715_amd import binding as B
from paper_2507_00715_amd.pipeline import EarnPath

DEV = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
ELEM = {"bf16": 2, "f32": 4}
ROPE_BASE = 10000.0


# ----------------------------------------------------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # The smallest request: two short prompts, fp32 (the precise form), prefill through every layer and the first
        # decode step with one call per layer.  Launches and latency, hardly any arithmetic.
        {"name": "path_small_f32", "kind": "path", "dtype": "f32", "batch": 2, "min_len": 100, "max_len": 132,
         "lengths": "uniform", "lengths_seed": 1, "h": 2, "t": 2, "layers": 4, "split_k": 2, "hq": 4, "hkv": 4, "d": 64,
         "beams": 1, "gen_cap": 4},
        # A serving batch of many short, log-uniformly spread histories: prefill of the full layers, compaction of the
        # register rows, the register-focused layers, and the first decode step.
        {"name": "path_serving", "kind": "path", "dtype": "bf16", "batch": 256, "min_len": 80, "max_len": 1040,
         "lengths": "loguniform", "lengths_seed": 2, "h": 8, "t": 8, "layers": 28, "split_k": 2, "hq": 12, "hkv": 2,
         "d": 128, "beams": 1, "gen_cap": 4},
        # One full-length layer over a ragged batch of medium prompts, multi-head, with attention sinks (a few keys eight
        # times as large).
        {"name": "prefill_ragged", "kind": "prefill", "dtype": "bf16", "batch": 64, "min_len": 288, "max_len": 2080,
         "lengths": "uniform", "lengths_seed": 3, "hq": 32, "hkv": 32, "d": 128, "outliers": 0.05},
        # One full-length layer over long prompts, grouped heads: the largest single call.
        {"name": "prefill_long", "kind": "prefill", "dtype": "bf16", "batch": 16, "min_len": 8256, "max_len": 8256,
         "lengths": "uniform", "lengths_seed": 4, "hq": 32, "hkv": 8, "d": 128, "outliers": 0.0},
        # One generated token through all layers of a small grouped-query model: a chain of small launches.
        {"name": "decode_small", "kind": "decode", "dtype": "bf16", "batch": 32, "min_len": 272, "max_len": 528,
         "lengths": "uniform", "lengths_seed": 5, "h": 8, "t": 8, "layers": 24, "split_k": 4, "hq": 14, "hkv": 2, "d": 64,
         "beams": 1, "gen_cap": 16, "step": 7},
        # The same with long prompts and ten beams per sequence that share its caches.
        {"name": "decode_long_beams", "kind": "decode", "dtype": "bf16", "batch": 16, "min_len": 8256, "max_len": 8256,
         "lengths": "uniform", "lengths_seed": 6, "h": 32, "t": 32, "layers": 32, "split_k": 4, "hq": 32, "hkv": 8,
         "d": 128, "beams": 10, "gen_cap": 8, "step": 3},
        # The same for a multi-head model over medium, ragged prompts: the most cache bytes per token.
        {"name": "decode_mha", "kind": "decode", "dtype": "bf16", "batch": 64, "min_len": 288, "max_len": 2080,
         "lengths": "uniform", "lengths_seed": 7, "h": 16, "t": 16, "layers": 32, "split_k": 8, "hq": 32, "hkv": 32,
         "d": 128, "beams": 1, "gen_cap": 8, "step": 3},
        # Beam search between two decode steps at beam width 20 over a language model's vocabulary: selection, ancestor
        # table, and the next step's attention through the table in one full-cache and one register-cache layer.
        {"name": "beam_step", "kind": "beam", "dtype": "bf16", "batch": 16, "min_len": 8256, "max_len": 8256,
         "lengths": "uniform", "lengths_seed": 8, "r": 64, "hq": 32, "hkv": 8, "d": 128, "beams": 20, "vocab": 32000,
         "gen_cap": 8, "step": 4},
        # The dense products of one decoder layer (Q/K/V with rotation, output, feed-forward) at the rows of two long
        # prompts, and at the rows of a decode step, where the weights' bytes are what moves.
        {"name": "projections_prefill", "kind": "projections", "rows": 16512, "d_model": 4096, "d_ffn": 11008, "hq": 32,
         "hkv": 8, "d": 128},
        {"name": "projections_decode", "kind": "projections", "rows": 160, "d_model": 4096, "d_ffn": 11008, "hq": 32,
         "hkv": 8, "d": 128},
        # The attention of a training step, forward and backward: a full-length layer over medium prompts, and a
        # register-focused layer, whose sequences are the registers and the target tokens.
        {"name": "train_full", "kind": "train", "dtype": "bf16", "batch": 16, "min_len": 272, "max_len": 1040,
         "lengths": "uniform", "lengths_seed": 9, "hq": 32, "hkv": 8, "d": 128},
        {"name": "train_registers", "kind": "train", "dtype": "bf16", "batch": 64, "min_len": 68, "max_len": 68,
         "lengths": "uniform", "lengths_seed": 10, "hq": 32, "hkv": 8, "d": 128},
    ]


# head counts and head dimensions of the configurations
HEADS = [(14, 2, 64), (32, 32, 128), (32, 8, 128), (12, 2, 128), (8, 8, 128), (4, 4, 64)]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _lengths_of(rng, case, lo, hi):
    longest = _log(rng, lo, hi)
    case.update(max_len=longest, min_len=max(lo, min(longest, int(longest * rng.uniform(0.1, 1.0)))),
                lengths=rng.choice(["uniform", "loguniform"]), lengths_seed=rng.randrange(1 << 30))


def draw(rng):
    kind = rng.choice(["path", "prefill", "decode", "beam", "projections", "train"])
    hq, hkv, d = rng.choice(HEADS)
    case = {"kind": kind, "hq": hq, "hkv": hkv, "d": d}
    if kind == "projections":
        case.update(d_model=hq * d, d_ffn=11008 if hq * d == 4096 else (int(hq * d * 2.6875) + 63) // 64 * 64)
        case["rows"] = _log(rng, 1, 16512)
        return case
    case["dtype"] = "f32" if kind in ("path", "prefill", "decode", "train") and rng.random() < 0.15 else "bf16"
    f32 = case["dtype"] == "f32"
    case["batch"] = _log(rng, 1, 16 if f32 else 256)
    if kind in ("path", "decode"):
        case.update(h=_log(rng, 1, 32), t=_log(rng, 1, 32), layers=rng.randint(4, 32), beams=rng.choice([1, 1, 1, 4, 10]))
        case["split_k"] = max(1, case["layers"] // rng.choice([4, 6, 8, 14]))
        case["gen_cap"] = rng.choice([4, 8, 16])
        if kind == "decode":
            case["step"] = rng.randrange(case["gen_cap"])
        _lengths_of(rng, case, case["h"] + case["t"], 512 if f32 else (2080 if kind == "path" else 8256))
        limit = {"bytes": 6e9, "flops": 3e12, "tokens": 60000 * 28 * 4096}
    elif kind == "prefill":
        case["outliers"] = rng.choice([0.0, 0.05])
        _lengths_of(rng, case, 33, 512 if f32 else 8256)
        limit = {"bytes": 6e9, "flops": 8.5e12, "tokens": 4e10}
    elif kind == "beam":
        case.update(r=_log(rng, 2, 64), beams=rng.randint(2, 20), vocab=_log(rng, 256, 32000), gen_cap=rng.choice([4, 8, 16]))
        case["step"] = rng.randrange(1, case["gen_cap"])
        case["batch"] = min(case["batch"], 64)
        _lengths_of(rng, case, 64, 8256)
        limit = {"bytes": 3e9, "flops": 3e12, "tokens": 4e10}
    else:
        _lengths_of(rng, case, 8, 256 if f32 else 2080)
        limit = {"bytes": 3e9, "flops": work(listed()[10])["flops"], "tokens": 4e10}
    # a drawn case costs no more than the largest listed one of its kind: fewer sequences until it does
    while case["batch"] > 1:
        w = work(case)
        tokens = sum(_lengths(case)) * case.get("layers", 1) * (hq + 2 * hkv) * d * 2
        if w["bytes"] <= limit["bytes"] and w["flops"] <= limit["flops"] * (0.02 if f32 else 1.0) and tokens <= limit["tokens"]:
            break
        case["batch"] = max(1, case["batch"] // 2)
    return case


# ----------------------------------------------------------------------------------------------------------------------
# sizes and work
# ----------------------------------------------------------------------------------------------------------------------
def _lengths(case):
    rng = random.Random(case["lengths_seed"])
    lo, hi = case["min_len"], case["max_len"]
    if case["lengths"] == "uniform":
        return [rng.randint(lo, hi) for _ in range(case["batch"])]
    return [min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))) for _ in range(case["batch"])]


def _prefill_work(case, lens, copies_keys=True):
    """bytes and flops of one layer's causal attention: q, k, v read, the output (and the rotated keys) written."""
    e, total = ELEM[case["dtype"]], sum(lens)
    pairs = sum(n * (n + 1) // 2 for n in lens)
    return (e * total * case["d"] * (2 * case["hq"] + (3 if copies_keys else 2) * case["hkv"]), 4 * case["d"] * case["hq"] * pairs)


def _decode_work(case, lens, step):
    """bytes and flops of one layer's decode step: shared rows once per sequence, generated rows per stream."""
    e, row = ELEM[case["dtype"]], case["hkv"] * case["d"]
    streams = case["batch"] * case["beams"]
    nbytes = e * (2 * row * (sum(lens) + streams * (step + 2)) + 2 * streams * case["hq"] * case["d"])
    keys = case["beams"] * sum(lens) + streams * (step + 1)
    return nbytes, 4 * case["d"] * case["hq"] * keys


def work(case):
    kind = case["kind"]
    if kind == "projections":
        r, dm, df, n = case["rows"], case["d_model"], case["d_ffn"], (case["hq"] + 2 * case["hkv"]) * case["d"]
        o = case["hq"] * case["d"]
        products = [(dm, n), (o, dm), (dm, df), (df, dm)]
        return {"bytes": 2 * sum(k * m + r * (k + m) for k, m in products), "flops": 2 * r * sum(k * m for k, m in products)}
    lens = _lengths(case)
    if kind == "prefill":
        nbytes, flops = _prefill_work(case, lens)
    elif kind == "train":
        # forward: q, k, v -> out, lse; backward: q, k, v, out, lse, d_out -> dq, dk, dv; five products instead of two
        nbytes, flops = _prefill_work(case, lens, copies_keys=False)
        e, total = ELEM[case["dtype"]], sum(lens)
        nbytes += total * (e * case["d"] * (4 * case["hq"] + 4 * case["hkv"]) + 8 * case["hq"])
        flops = flops * 7 // 2
    else:
        nbytes = flops = 0
        k = case.get("split_k", 1)
        rest = case["layers"] - k if kind != "beam" else 1
        regs = [case["r"] if kind == "beam" else case["h"] + case["t"]] * case["batch"]
        if kind == "path":
            for layers, ln in ((k, lens), (rest, regs)):
                b, f = _prefill_work(case, ln)
                nbytes, flops = nbytes + layers * b, flops + layers * f
            # the compaction: the hidden rows and the later layers' q, k, v, read and written
            cols = case["hq"] * case["d"] + rest * (case["hq"] + 2 * case["hkv"]) * case["d"]
            nbytes += 2 * ELEM[case["dtype"]] * sum(regs) * cols
        for layers, ln in ((k, lens), (rest, regs)):
            b, f = _decode_work(case, ln, case.get("step", 0))
            nbytes, flops = nbytes + layers * b, flops + layers * f
        if kind == "beam":
            nbytes += 4 * case["batch"] * case["beams"] * (case["vocab"] + 3 + 2 * case["gen_cap"])
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the errors measured against the same functions in 64 bits (relative 2-norm; largest difference
    over the result's root mean square): fp32 7e-7 and 5e-6; bf16 prefill 4e-3 and 6e-2, with large keys 5e-3 and 9e-2
    (a rounded operand moves a large key's score in proportion); decode 3e-3 and 1e-2; products 3e-3 and 1.4e-2;
    gradients 2.5e-3 and 5e-2.  Selected tokens, tables and row indices are whole numbers and do not differ."""
    if case.get("dtype") == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    rel, largest = {"path": (1.6e-2, 0.25), "prefill": (1.6e-2, 0.25), "decode": (1.2e-2, 0.06), "beam": (1.2e-2, 0.06),
                    "projections": (1.2e-2, 0.06), "train": (1e-2, 0.2)}[case["kind"]]
    return {"rel": 2e-2, "max": 0.4} if case.get("outliers", 0.0) > 0.0 else {"rel": rel, "max": largest}


# ----------------------------------------------------------------------------------------------------------------------
# what a program has in hand
# ----------------------------------------------------------------------------------------------------------------------
class _Inputs:
    def __init__(self, case, seed):
        self.g = torch.Generator(device=DEV).manual_seed(seed)
        self.dtype = DTYPES[case.get("dtype", "bf16")]

    def randn(self, *shape, scale=1.0):
        x = torch.randn(shape, generator=self.g, device=DEV, dtype=self.dtype)
        return x.mul_(scale) if scale != 1.0 else x

    def keys(self, outliers, *shape):
        k = self.randn(*shape)
        if outliers > 0.0:
            k.mul_(1.0 + 7.0 * (torch.rand(shape[:2], generator=self.g, device=DEV) < outliers).to(k.dtype)[:, :, None])
        return k


def _i32(values):
    return torch.tensor(list(values), dtype=torch.int32, device=DEV)


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return cu


def _desc(case, rope_base=ROPE_BASE):
    return B.make_desc(DTYPES[case.get("dtype", "bf16")], case["hq"], case["hkv"], case["d"], 0.0, rope_base)


def _buffer(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def _earn_path(case, lens):
    return EarnPath(n_layers=case["layers"], split_k=case["split_k"], n_head_reg=case["h"], n_tail_reg=case["t"],
                    n_q_heads=case["hq"], n_kv_heads=case["hkv"], head_dim=case["d"], dtype=DTYPES[case["dtype"]],
                    cu_seqlens=_cu(lens), stream_to_seq=[s for s in range(case["batch"]) for _ in range(case["beams"])],
                    gen_cap=case["gen_cap"], rope_base=ROPE_BASE, device=DEV)


def prepare(case, seed):
    return {"path": _prepare_path, "prefill": _prepare_prefill, "decode": _prepare_decode, "beam": _prepare_beam,
            "projections": _prepare_projections, "train": _prepare_train}[case["kind"]](case, _Inputs(case, seed))


def run(state):
    return {"path": _run_path, "prefill": _run_prefill, "decode": _run_decode, "beam": _run_beam,
            "projections": _run_projections, "train": _run_train}[state["kind"]](state)


# ---- a request batch through the whole path: prefill of all layers, then the first decode step ----
def _prepare_path(case, x):
    lens = _lengths(case)
    n, total, streams = case["layers"], sum(lens), case["batch"] * case["beams"]
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    s = {"kind": "path", "path": _earn_path(case, lens), "x": x.randn(total, hq * d)}
    s["q"], s["k"], s["v"] = ([x.randn(total, heads, d) for _ in range(n)] for heads in (hq, hkv, hkv))
    s["dq"], s["dk"], s["dv"] = (x.randn(n, streams, heads, d) for heads in (hq, hkv, hkv))
    return s


def _run_path(s):
    p = s["path"]
    p.prefill(s["q"], s["k"], s["v"], s["x"])
    p.decode_step(0, s["dq"], s["dk"], s["dv"])
    return {"full": p.prefill_out[:p.k], "registers": p.reg_prefill_out, "full_keys": p.full_k_cache,
            "register_keys": p.reg_k_cache, "register_values": p.reg_v, "hidden": p.x_c, "rows": p.idx, "positions": p.pos,
            "decode": p.decode_out_all, "generated_keys": p.gen_k_all, "generated_values": p.gen_v_all}


# ---- one full-length layer, the rotated keys kept as its cache ----
def _prepare_prefill(case, x):
    lens = _lengths(case)
    total, hq, hkv, d = sum(lens), case["hq"], case["hkv"], case["d"]
    s = {"kind": "prefill", "desc": _desc(case), "cu": _i32(_cu(lens)), "batch": case["batch"], "total": total,
         "longest": max(lens), "q": x.randn(total, hq, d), "k": x.keys(case["outliers"], total, hkv, d),
         "v": x.randn(total, hkv, d)}
    s["out"], s["k_rot"] = torch.empty_like(s["q"]), torch.empty_like(s["k"])
    s["workspace"] = _buffer(B.earn_prefill_workspace_bytes(s["desc"], case["batch"], total, s["longest"], True))
    return s


def _run_prefill(s):
    B.earn_prefill_attn(s["desc"], s["q"], s["k"], s["v"], s["cu"], None, s["batch"], s["total"], s["longest"], s["out"],
                        s["k_rot"], None, s["workspace"])
    return s["out"], s["k_rot"]


# ---- one decode step through all layers, one call per layer bound to its buffers (layer l + 1 needs layer l) ----
def _prepare_decode(case, x):
    lens = _lengths(case)
    p = _earn_path(case, lens)
    streams, hq, hkv, d, step = case["batch"] * case["beams"], case["hq"], case["hkv"], case["d"], case["step"]
    for cache in (p.full_k_cache, p.reg_k_cache, p.reg_v, p.gen_k_all, p.gen_v_all):
        cache.normal_(generator=x.g)
    values = x.randn(p.k, p.T, hkv, d)
    for l in range(p.N):
        p.v_cache[l] = values[l] if l < p.k else p.v_c[l]
    q, k, v = (x.randn(p.N, streams, heads, d) for heads in (hq, hkv, hkv))
    calls = [p.bind_set_step(step)] + [p.bind_decode_layer(l, q[l], k[l], v[l]) for l in range(p.N)]
    return {"kind": "decode", "path": p, "calls": calls}


def _run_decode(s):
    for call in s["calls"]:
        call()
    p = s["path"]
    return p.decode_out_all, p.gen_k_all, p.gen_v_all


# ---- beam search: selection, ancestor table, the next step's attention through it ----
def _prepare_beam(case, x):
    lens, beams, g = _lengths(case), case["beams"], case["step"]
    streams, hq, hkv, d, cap = case["batch"] * beams, case["hq"], case["hkv"], case["d"], case["gen_cap"]
    e = lambda *shape, dtype=torch.int32: torch.empty(shape, dtype=dtype, device=DEV)
    desc = _desc(case)
    s = {"kind": "beam", "desc": desc, "batch": case["batch"], "beams": beams, "vocab": case["vocab"], "streams": streams,
         "cap": cap, "step": g, "stream_to_seq": _i32(u // beams for u in range(streams)),
         "scores": -4.0 * torch.rand(streams, generator=x.g, device=DEV),
         "logp": torch.log_softmax(torch.randn(streams, case["vocab"], generator=x.g, device=DEV) * 2.0, dim=-1),
         "parent": e(streams), "token": e(streams), "new_scores": e(streams, dtype=torch.float32),
         "table": e(streams, cap), "gen_len": _i32([g] * streams)}
    own = torch.arange(streams, dtype=torch.int32, device=DEV)[:, None] // beams * beams
    s["old_table"] = (torch.randint(0, beams, (streams, cap), generator=x.g, device=DEV, dtype=torch.int32) + own).contiguous()
    s["q_pos"] = _i32(lens[u // beams] + g for u in range(streams))
    s["select_workspace"] = _buffer(B.earn_beam_topk_workspace_bytes(case["batch"], beams, case["vocab"]))
    s["layers"] = []
    for ln in (lens, [case["r"]] * case["batch"]):
        s["layers"].append({
            "cu": _i32(_cu(ln)), "longest": max(ln), "k": x.randn(sum(ln), hkv, d), "v": x.randn(sum(ln), hkv, d),
            "q": x.randn(streams, hq, d), "k_new": x.randn(streams, hkv, d), "v_new": x.randn(streams, hkv, d),
            "gen_k": x.randn(streams, cap, hkv, d), "gen_v": x.randn(streams, cap, hkv, d),
            "out": torch.empty(streams, hq, d, dtype=x.dtype, device=DEV),
            "workspace": _buffer(B.earn_decode_workspace_bytes(desc, streams, case["batch"], max(ln), cap))})
    return s


def _run_beam(s):
    B.earn_beam_topk(s["scores"], s["logp"], s["batch"], s["beams"], s["vocab"], s["parent"], s["token"], s["new_scores"],
                     s["select_workspace"])
    B.earn_beam_reorder(s["parent"], s["old_table"], s["table"], s["streams"], s["cap"], s["step"] - 1)
    for l in s["layers"]:
        B.earn_decode_attn_beams(s["desc"], l["q"], l["k_new"], l["v_new"], s["q_pos"], l["k"], l["v"], l["cu"],
                                 s["stream_to_seq"], l["gen_k"], l["gen_v"], s["gen_len"], s["table"], s["cap"],
                                 s["streams"], s["batch"], l["longest"], l["out"], l["workspace"])
    return {"parent": s["parent"], "token": s["token"], "scores": s["new_scores"], "table": s["table"],
            "layers": [[l["out"], l["gen_k"], l["gen_v"]] for l in s["layers"]]}


# ---- the dense products of one decoder layer ----
def _prepare_projections(case, x):
    rows, dm, df, hq, hkv, d = (case[k] for k in ("rows", "d_model", "d_ffn", "hq", "hkv", "d"))
    e = lambda *shape: torch.empty(shape, dtype=x.dtype, device=DEV)
    s = {"kind": "projections", "desc": _desc(case), "x": x.randn(rows, dm), "attended": x.randn(rows, hq * d),
         "w_qkv": x.randn((hq + 2 * hkv) * d, dm, scale=dm ** -0.5), "w_o": x.randn(dm, hq * d, scale=(hq * d) ** -0.5),
         "w_up": x.randn(df, dm, scale=dm ** -0.5), "w_down": x.randn(dm, df, scale=df ** -0.5),
         "positions": torch.randint(0, 8256, (rows,), generator=x.g, device=DEV, dtype=torch.int32),
         "q": e(rows, hq, d), "k": e(rows, hkv, d), "v": e(rows, hkv, d), "y": e(rows, dm), "hidden": e(rows, df),
         "z": e(rows, dm)}
    s["workspace"] = _buffer(max(B.earn_linear_workspace_bytes(rows, k, n) for k, n in
                                 ((dm, (hq + 2 * hkv) * d), (hq * d, dm), (dm, df), (df, dm))))
    return s


def _run_projections(s):
    ws = s["workspace"]
    B.earn_qkv_rope_project(s["desc"], s["x"], s["w_qkv"], None, s["positions"], 1, s["q"], s["k"], s["v"], ws)
    B.earn_linear(s["attended"], s["w_o"], s["y"], 0, ws)
    B.earn_linear(s["y"], s["w_up"], s["hidden"], 1, ws)
    B.earn_linear(s["hidden"], s["w_down"], s["z"], 0, ws)
    return s["q"], s["k"], s["v"], s["y"], s["hidden"], s["z"]


# ---- the attention of a training step: forward with its log-sum-exp, then the gradients ----
def _prepare_train(case, x):
    lens = _lengths(case)
    total, hq, hkv, d = sum(lens), case["hq"], case["hkv"], case["d"]
    s = {"kind": "train", "desc": _desc(case, 0.0), "cu": _i32(_cu(lens)), "batch": case["batch"], "total": total,
         "longest": max(lens), "q": x.randn(total, hq, d), "k": x.randn(total, hkv, d), "v": x.randn(total, hkv, d),
         "d_out": x.randn(total, hq, d), "lse": torch.empty(total, hq, dtype=torch.float32, device=DEV)}
    for grad, of in (("out", "q"), ("dq", "q"), ("dk", "k"), ("dv", "v")):
        s[grad] = torch.empty_like(s[of])
    return s


def _run_train(s):
    B.earn_prefill_attn(s["desc"], s["q"], s["k"], s["v"], s["cu"], None, s["batch"], s["total"], s["longest"], s["out"],
                        None, s["lse"], None)
    B.earn_attn_backward(s["desc"], s["q"], s["k"], s["v"], s["out"], s["lse"], s["d_out"], s["cu"], s["batch"], s["total"],
                         s["longest"], s["dq"], s["dk"], s["dv"])
    return s["out"], s["lse"], s["dq"], s["dk"], s["dv"]
