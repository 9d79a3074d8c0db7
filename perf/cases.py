"""The work this library is timed on: training steps of the drafter's attention over the sequence lengths of the
training distribution (median 3,891, P90 10,800, P99 20,000 tokens), in each of the step's forms, and drafting
steps of the serving path.  Shapes are those of `peagle_inputs.CONFIGS`, of `bench.py` and of the tests; every case
goes through the public entry points of `paper_2602_01469_amd`.

A case is a dict of plain values; `kind` names the form of the call:

  step      one training step on a dense tile map (peagle_attn_step_partitioned, or _rope with a rotary base)
  separate  forward and backward as two calls over the whole sequence (what an autograd function does)
  shared    first-layer form (peagle_attn_step_rope_shared)
  sampled   a drop-token sampled sequence: new sample, map rebuilt in place, training step
  packed    several sequences of different lengths as one problem
  draft     one drafting step against a paged cache
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2602_01469_amd as pe
from peagle_inputs import CONFIGS, PAGE_TOKENS, cod_depth_counts, useful_pairs

ROPE_BASE = 500000.0
RETENTION = 0.8           # the paper's training setting of drop-token sampling
HEADS = {64: (64, 8), 128: (32, 4)}  # query / KV heads of the two drafter shapes
LARGEST_FLOPS = 1.0e14    # no drawn case does more than the largest listed one


def _config(config, **more):
    c = CONFIGS[config]
    case = {"kind": "step", "L": c.L, "L_max": c.L, "K": c.K, "Hq": c.Hq, "Hkv": c.Hkv, "D": c.D, "seg": c.seg_anchors,
            "value_scale": c.value_scale, "rope": False, "grad_bf16": False}
    case.update(more)
    return case


def _draft(C, K, D, ctx_lo, ctx_hi, graph):
    Hq, Hkv = HEADS[D]
    return {"kind": "draft", "C": C, "K": K, "Hq": Hq, "Hkv": Hkv, "D": D, "ctx_lo": ctx_lo, "ctx_hi": ctx_hi,
            "graph": graph}


def listed():
    return [
        # The smallest training call: a short prompt on a small drafter; launches and host time count.
        _config("c1_tiny", name="step_tiny"),
        # A short example of the training distribution (its 0.1 quantile, ragged) on the one map that a training
        # program builds for its longest sequence: prefix view, cropped segment.
        _config("c3_median", name="step_short_prefix", L=1391, L_max=8192, seg=2048),
        # Forward and backward called apart, over the whole sequence, as an autograd function calls them.
        _config("c2_gptoss", name="separate_calls", kind="separate"),
        # The headline: the median length of the training distribution, four segments.
        _config("c3_median", name="step_median"),
        # The P90 length on the larger head size, rotary embedding inside, gradients rounded to bf16 for the optimizer.
        _config("c4_p90", name="step_p90_rope_d128", rope=True, grad_bf16=True),
        # The P99 length: the longest sequence that the paper trains on, ten segments.
        _config("c5_p99", name="step_p99"),
        # The first drafter layer at the paper's exact median length (odd): shared key / value vector.
        _config("c3_median", name="shared_median", kind="shared", L=3891, L_max=3891, rope=True),
        # The production training setting: 8192 tokens, K = 8, retention 0.8; each example has a new sample.
        _config("c3_median", name="sampled_8k", kind="sampled", L=8192, L_max=8192, seg=2048),
        # Short examples packed into one problem (an odd mixture of lengths).
        _config("c3_median", name="packed_short", kind="packed", L=6420, L_max=6420, seg=0,
                lens="1248 203 517 1456 64 871 333 1728"),
        # Serving: four requests, seven draft positions, replayed from a graph as a serving loop does.
        _draft(4, 7, 64, 2048, 4096, True) | {"name": "draft_serving_graph"},
        # Serving: two requests with long contexts, larger heads, called directly.
        _draft(2, 5, 128, 10800, 20000, False) | {"name": "draft_long_d128"},
        # A full batch of requests of all lengths: the cache read fills the memory system.
        _draft(64, 7, 64, 512, 8192, False) | {"name": "draft_batch"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _segment(rng, L, K):
    """Anchors per segment: a whole number of row tiles (128 / K anchors), or one segment."""
    A = 128 // K
    want = rng.choice([0, 1024, 2048])
    return 0 if want == 0 or want >= L else max(1, want // A) * A


def draw(rng):
    kind = rng.choice(["step", "step", "step", "separate", "shared", "sampled", "packed", "draft", "draft", "draft"])
    D = rng.choice([64, 64, 128])
    if kind == "draft":
        C = _log_int(rng, 1, 64)
        hi = _log_int(rng, 256, 20000 if C <= 16 else 8192)
        return _draft(C, rng.choice([3, 4, 5, 7, 8]), D, max(1, int(hi * rng.uniform(0.1, 1.0))), hi, rng.random() < 0.5)
    Hq, Hkv = HEADS[D] if rng.random() < 0.8 else (4, 1)
    K = rng.choice([4, 5, 7, 8, 8, 8])
    case = {"kind": kind, "K": K, "Hq": Hq, "Hkv": Hkv, "D": D, "value_scale": rng.choice([0.5, 1.0]),
            "rope": kind in ("step", "shared") and (kind == "shared" or rng.random() < 0.4),
            "grad_bf16": kind in ("step", "sampled") and rng.random() < 0.4}
    if kind == "packed":
        lens = [_log_int(rng, 48, 4096) for _ in range(rng.randint(2, 12))]
        return case | {"L": sum(lens), "L_max": sum(lens), "seg": 0, "lens": " ".join(map(str, lens))}
    L = _log_int(rng, 128, 20480 if kind != "separate" else 8192)
    L_max = L if kind != "step" or rng.random() < 0.5 else min(20480, int(L * rng.uniform(1.0, 2.0)))
    case |= {"L": L, "L_max": L_max, "seg": 0 if kind == "separate" else _segment(rng, L_max, K)}
    assert work(case)["flops"] <= LARGEST_FLOPS
    return case


# ------------------------------------------------------------------------------------------ sizes

def _depths(case, seed):
    return cod_depth_counts(case["L"], case["K"], RETENTION, seed)


def _bounds(case):
    L, seg = case["L_max"], case["seg"]
    return list(range(0, L, seg)) + [L] if seg else [0, L]


def _lens(case):
    return [int(x) for x in case["lens"].split()]


def _contexts(case):
    """Context lengths of the requests of a batch: from ctx_lo to ctx_hi, the longest always present, in a mixed order."""
    C, lo, hi = case["C"], case["ctx_lo"], case["ctx_hi"]
    lens = [hi] if C == 1 else [lo + (hi - lo) * i // (C - 1) for i in range(C)]
    random.Random(C * 1000003 + hi).shuffle(lens)
    return lens


def _tokens_and_pairs(case):
    """Stored tokens, and visible (row, key) pairs per query head."""
    K = case["K"]
    if case["kind"] == "packed":
        return sum(_lens(case)) * K, sum(useful_pairs(n, K) for n in _lens(case))
    if case["kind"] == "sampled":  # (the counts per depth do not depend on the draw; the pairs hardly do)
        n = _depths(case, 0).astype(np.int64)
        return int(n.sum()), int((n * (np.arange(len(n)) + 1) + n * (n - 1) // 2).sum())
    return case["L"] * K, useful_pairs(case["L"], K)


def work(case):
    Hq, Hkv, D, K = case["Hq"], case["Hkv"], case["D"], case["K"]
    if case["kind"] == "draft":
        ctx, rows = _contexts(case), case["C"] * K
        return {"bytes": 2 * sum(ctx) * Hkv * D * 2 + 2 * rows * Hq * D * 2 + 2 * rows * Hkv * D * 2 + rows * Hq * 4,
                "flops": 4 * D * Hq * sum(K * n + K * (K + 1) // 2 for n in ctx)}
    T, pairs = _tokens_and_pairs(case)
    keys = case["L"] if case["kind"] == "shared" else T  # K, V rows in, dK, dV rows out
    out = 4 + (2 if case["grad_bf16"] else 0)            # bytes per element of dK, dV
    return {"bytes": 4 * T * Hq * D * 2 + 2 * keys * Hkv * D * (2 + out) + T * Hq * 4, "flops": 14 * D * Hq * pairs}


def tolerance(case):
    """bf16 operands and outputs; probabilities and dS are rounded to bf16 before they enter a matrix product.  Against
    the same computation in 64 bits O is off by 2.2e-3 in norm and the gradients by 1.7e-3 to 2.6e-3 (rotary: one more
    rounding of Q and K, 2.7e-3 to 3.6e-3); single elements, in rows whose weight sits on a few keys, by up to 0.22 of
    the tensor's rms (rotary 0.31).  About four times that; a drafting step's rows see many keys."""
    if case["kind"] == "draft":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 1.4e-2, "max": 0.95} if case["rope"] else {"rel": 1e-2, "max": 0.85}


# ----------------------------------------------------------------------------------------- states

def _tensors(case, T, g):
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    rnd = lambda *sh: (torch.randn(*sh, generator=g, device="cuda") * case["value_scale"]).to(torch.bfloat16)
    keys = case["L"] if case["kind"] == "shared" else T
    s = {"q": rnd(T, Hq, D), "k": rnd(keys, Hkv, D), "v": rnd(keys, Hkv, D), "d_o": rnd(T, Hq, D)}
    s["o"], s["dq"] = torch.empty_like(s["q"]), torch.empty_like(s["q"])
    s["lse"] = torch.empty((Hq, T), device="cuda")
    s["dk"], s["dv"] = (torch.empty((keys, Hkv, D), device="cuda") for _ in range(2))
    s["dk16"], s["dv16"] = (torch.empty_like(s["k"]) for _ in range(2)) if case["grad_bf16"] else (None, None)
    if case["kind"] == "shared":
        s["k_shared"], s["v_shared"] = rnd(Hkv, D), rnd(Hkv, D)
        s["dk_shared"], s["dv_shared"] = (torch.empty((Hkv, D), device="cuda") for _ in range(2))
    return s


def _prepare_draft(case, g):
    C, K, Hq, Hkv, D = case["C"], case["K"], case["Hq"], case["Hkv"], case["D"]
    ctx = _contexts(case)
    pages = [(n + PAGE_TOKENS - 1) // PAGE_TOKENS for n in ctx]
    n_pages, max_pages = sum(pages), max(pages)
    rnd = lambda *sh: torch.randn(*sh, generator=g, device="cuda").to(torch.bfloat16)
    s = {"q": rnd(C, K, Hq, D), "k": rnd(C, K, Hkv, D), "v": rnd(C, K, Hkv, D),
         "k_pages": rnd(n_pages, Hkv, PAGE_TOKENS, D), "v_pages": rnd(n_pages, Hkv, PAGE_TOKENS, D)}
    perm = torch.randperm(n_pages, generator=g, device="cuda").to(torch.int32)  # a pool in use: pages in any order
    table = torch.full((C, max_pages), -1, dtype=torch.int32, device="cuda")
    at = 0
    for c, n in enumerate(pages):
        table[c, :n] = perm[at:at + n]
        at += n
    s["table"], s["ctx"] = table, torch.tensor(ctx, dtype=torch.int32, device="cuda")
    s["o"], s["lse"] = torch.empty_like(s["q"]), torch.empty((C, Hq, K), device="cuda")
    s["status"] = torch.empty((C,), dtype=torch.int32, device="cuda")
    s["shape"] = pe.DecodeShape(C, K, Hq, Hkv, D, n_pages, max_pages)
    s["ws"] = torch.empty(pe.peagle_draft_decode_workspace_bytes(s["shape"]), dtype=torch.uint8, device="cuda")
    s["graph"] = None
    if case["graph"]:  # recorded once per shape and set of buffers
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _call_draft(s)
        s["graph"] = graph
    return s


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    if case["kind"] == "draft":
        return _prepare_draft(case, g) | {"case": case}
    L, K, kind, depths = case["L"], case["K"], case["kind"], None
    if kind == "packed":
        tm = pe.peagle_build_tilemap_packed(_lens(case), K)
    elif kind == "sampled":
        depths = _depths(case, seed)
        tm = pe.peagle_build_tilemap_sampled(_depths(case, seed + 1), K, _bounds(case))  # an earlier example's sample
    else:
        tm = pe.peagle_build_tilemap(case["L_max"], K, _bounds(case))
    shape = pe.Shape(L if kind != "packed" else sum(_lens(case)), K, case["Hq"], case["Hkv"], case["D"])
    s = _tensors(case, tm.tokens(shape.L), g)
    s |= {"case": case, "tm": tm, "shape": shape, "depths": depths, "bounds": _bounds(case) if kind != "packed" else None}
    s["S"] = 1 if kind == "packed" else len(s["bounds"]) - 1
    need = pe.peagle_workspace_bytes
    if case["rope"]:
        n_pos = pe.peagle_rope_positions(tm, shape.L)
        s["table"] = torch.empty((n_pos, 2, case["D"] // 2), device="cuda")
        pe.peagle_rope_table(ROPE_BASE, case["D"], n_pos, s["table"])
        need = pe.peagle_rope_shared_workspace_bytes if kind == "shared" else pe.peagle_rope_workspace_bytes
    s["ws"] = torch.empty(need(tm, shape), dtype=torch.uint8, device="cuda")
    return s


# ------------------------------------------------------------------------------------------- runs

def _call_draft(s):
    pe.peagle_draft_decode(s["shape"], s["q"], s["k"], s["v"], s["k_pages"], s["v_pages"], s["table"], s["ctx"], s["o"],
                           s["lse"], s["status"], s["ws"])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "draft":
        if s["graph"] is not None:
            s["graph"].replay()
        else:
            _call_draft(s)
        return {"o": s["o"], "lse": s["lse"], "status": s["status"]}
    out = {n: s[n] for n in ("o", "lse", "dq", "dk", "dv")}
    tm, shape = s["tm"], s["shape"]
    if kind == "separate":
        pe.peagle_attn_fwd(tm, shape, -1, s["q"], s["k"], s["v"], s["o"], s["lse"])
        pe.peagle_attn_bwd(tm, shape, -1, s["q"], s["k"], s["v"], s["o"], s["d_o"], s["lse"], s["dq"], s["dk"], s["dv"], 0,
                           s["ws"])
        return out
    if kind == "shared":
        pe.peagle_attn_step_rope_shared(tm, shape, s["q"], s["k"], s["k_shared"], s["v"], s["v_shared"], s["d_o"], s["table"],
                                        s["o"], s["lse"], s["dq"], s["dk"], s["dv"], s["dk_shared"], s["dv_shared"], s["ws"])
        return out | {"dk_shared": s["dk_shared"], "dv_shared": s["dv_shared"]}
    if kind == "sampled":  # every training example draws its own sample
        tm.rebuild([case["L"]], s["depths"], s["bounds"])
    if case["rope"]:
        pe.peagle_attn_step_partitioned_rope(tm, shape, 0, s["S"], s["q"], s["k"], s["v"], s["d_o"], s["table"], s["o"],
                                             s["lse"], s["dq"], s["dk"], s["dv"], s["dk16"], s["dv16"], s["ws"])
    else:
        pe.peagle_attn_step_partitioned(tm, shape, 0, s["S"], s["q"], s["k"], s["v"], s["d_o"], s["o"], s["lse"], s["dq"],
                                        s["dk"], s["dv"], s["dk16"], s["dv16"], s["ws"])
    if case["grad_bf16"]:
        out |= {"dk16": s["dk16"], "dv16": s["dv16"]}
    return out
