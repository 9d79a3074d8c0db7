"""GPU parity tests of the inference-side drafting attention (Sec. 2 of the paper: all K draft positions
of a request in one forward pass; serving shapes K = 3, 5, 7 at concurrency 2-4) against the fp64 oracle.
Tolerances are the forward's: O max-abs <= 1e-2 where bf16 allows / rel-L2 <= 5e-3, LSE <= 4e-3."""
import numpy as np
import pytest
import torch

import paper_2602_01469_amd as pe
from gpu_harness import bf16_to_f64, max_abs, rel_l2, to_dev_bf16
from oracle import peagle_oracle as orc
from peagle_inputs import bf16_bits_to_f64, f32_to_bf16_bits, make_decode_inputs
from test_gpu_parity import FWD_REL, LSE_ABS, _check_o_abs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


class DecodeRun:
    def __init__(self, inp, K, Hq, Hkv, D, scale=None, n_pages=None):
        C = len(inp["ctx_len"])
        self.shape = pe.DecodeShape(C, K, Hq, Hkv, D, n_pages or inp["n_pages"], inp["max_pages"], scale)
        self.q, self.k, self.v = (to_dev_bf16(inp[n]) for n in ("q_new", "k_new", "v_new"))
        self.kp, self.vp = to_dev_bf16(inp["k_pages"]), to_dev_bf16(inp["v_pages"])
        self.bt = torch.from_numpy(inp["block_table"]).cuda()
        self.cl = torch.from_numpy(inp["ctx_len"]).cuda()
        self.o = torch.full((C, K, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        self.lse = torch.full((C, Hq, K), float("nan"), dtype=torch.float32, device="cuda")
        self.status = torch.full((C,), -7, dtype=torch.int32, device="cuda")
        self.ws = torch.empty(pe.peagle_draft_decode_workspace_bytes(self.shape), dtype=torch.uint8, device="cuda")

    def run(self):
        pe.peagle_draft_decode(self.shape, self.q, self.k, self.v, self.kp, self.vp, self.bt, self.cl, self.o, self.lse,
                               self.status, self.ws)
        torch.cuda.synchronize()
        return bf16_to_f64(self.o), self.lse.double().cpu().numpy(), self.status.cpu().numpy()


def _oracle(inp, c, scale):
    f = bf16_bits_to_f64
    return orc.draft_decode(f(inp["q_new"][c]), f(inp["k_new"][c]), f(inp["v_new"][c]), f(inp["k_ctx"][c]),
                            f(inp["v_ctx"][c]), scale)


def _check(inp, o, lse, scale, what):
    assert not np.isnan(o).any() and not np.isnan(lse).any(), what
    for c in range(len(inp["ctx_len"])):
        ro, rl = _oracle(inp, c, scale)
        assert rel_l2(o[c], ro) <= FWD_REL, (what, c)
        _check_o_abs(o[c], ro, f"{what} request {c}")
        assert max_abs(lse[c], rl) <= LSE_ABS, (what, c)


def _form(shape):
    """(pieces, two wave groups?, requests ranked by length?) of a shape: the launcher's choice of kernel, on the pieces that
    it reports."""
    pieces = pe.peagle_draft_decode_splits(shape)
    wgs, long = shape.C * shape.Hkv * pieces, -(-shape.max_pages // pieces) > 16
    two = shape.K * (shape.Hq // shape.Hkv) <= 64 and (wgs <= 512 or long if shape.D == 64 else wgs <= 256)
    return pieces, two, 1 < shape.C <= 64 and wgs > 512 and long


DECODE = [
    # name, ctx_lens, K, Hq, Hkv, D, seed
    ("paper_c4_k7", (900, 1500, 333, 2048), 7, 64, 8, 64, 1000),
    ("paper_c2_k5", (700, 64), 5, 64, 8, 64, 1010),
    ("paper_c2_k3_d128", (513, 1200), 3, 32, 4, 128, 1020),
    ("page_edges", (0, 1, 63, 64, 65, 127, 128, 129), 4, 8, 2, 64, 1030),
    ("one_row_block", (300,), 3, 8, 1, 64, 1040),          # 24 rows: one wave
    ("four_row_blocks", (300, 10), 8, 16, 1, 64, 1050),    # 128 rows: four waves
    ("mha_k1_plain_decode", (500, 77), 1, 4, 4, 64, 1060),
    ("k7_d128_odd_group", (1000, 257, 5), 7, 9, 3, 128, 1070),
    ("long_context_many_splits", (20000, 4096), 7, 64, 8, 64, 1080),
    # 16 requests x 8 KV heads -> 8 context pieces; 131 block-table columns -> 17 pages per piece, in more than 512
    # workgroups: two wave groups, requests taken by falling length.  An odd tail, an empty request, one-page and
    # page-edge requests and K < 8 in the same batch.
    ("long_pieces_mixed_batch", (8371, 0, 77, 8257, 1000, 64, 8192, 3, 4097, 129, 0, 6000, 8384, 511, 2048, 65),
     5, 32, 8, 64, 1090),
]


@pytest.mark.parametrize("name,ctx_lens,K,Hq,Hkv,D,seed", DECODE, ids=[c[0] for c in DECODE])
def test_draft_decode_matches_oracle(name, ctx_lens, K, Hq, Hkv, D, seed):
    print(f"case decode {name}: ctx={ctx_lens} K={K} Hq={Hq} Hkv={Hkv} D={D} seed={seed}", flush=True)
    inp = make_decode_inputs(ctx_lens, K, Hq, Hkv, D, seed)
    r = DecodeRun(inp, K, Hq, Hkv, D)
    o, lse, status = r.run()
    assert (status == 0).all()
    _check(inp, o, lse, r.shape.scale, name)
    o2, lse2, _ = r.run()                                   # same buffers, same workspace: identical bits
    assert np.array_equal(o, o2) and np.array_equal(lse, lse2)
    if name == "long_pieces_mixed_batch":                   # the case exists to reach two wave groups and the ranking
        assert _form(r.shape) == (8, True, True)


def _with_probabilities_in_bf16(q, k, v, scale, pieces):
    """Attention of one query row in 64 bits but for what the kernel rounds: each piece's probabilities, relative to the
    largest score of its first 32 keys, and the output."""
    s = (k @ q) * (scale * np.log2(np.e))
    to_bf16 = lambda x: bf16_bits_to_f64(f32_to_bf16_bits(x.astype(np.float32)))
    m = [s[p[:32]].max() for p in pieces]
    ps = [to_bf16(np.exp2(s[p] - r)) for p, r in zip(pieces, m)]
    w = [2.0 ** (r - max(m)) for r in m]
    o = sum(x * (p @ v[i]) for x, p, i in zip(w, ps, pieces)) / sum(x * p.sum() for x, p in zip(w, ps))
    return to_bf16(o)


@pytest.mark.parametrize("D,ctx", [(64, 709), (128, 500)])
def test_draft_decode_in_one_piece_is_no_less_exact_than_in_pieces_of_four_pages(D, ctx):
    """A key whose score is the reference maximum has the probability 1, without rounding, and in rows of few heavy keys that
    counts: every four pages used to start two references (two wave groups that take the pages in turn).  One piece for all
    pages must not be further from 64 bits than that."""
    C, K, Hkv = 4, 5, 4
    Hq = 8 * Hkv
    print(f"case decode exactness D={D} ctx={ctx}", flush=True)
    inp = make_decode_inputs((ctx,) * C, K, Hq, Hkv, D, 1500 + D)
    r = DecodeRun(inp, K, Hq, Hkv, D)
    assert pe.peagle_draft_decode_splits(r.shape) == 1
    o, _, _ = r.run()
    f = bf16_bits_to_f64
    pages = [np.arange(a, min(a + 64, ctx)) for a in range(0, ctx, 64)]
    err = {"one piece": 0.0, "four pages": 0.0}
    for c in range(C):
        ref, _ = _oracle(inp, c, r.shape.scale)
        k, v = (np.concatenate([f(inp[n + "_ctx"][c]), f(inp[n + "_new"][c])]) for n in ("k", "v"))
        for d in range(K):
            new = np.arange(ctx, ctx + d + 1)
            pieces = [np.concatenate(pages[a + g:a + 4:2] + ([new] if a + g == 0 else []))
                      for a in range(0, len(pages), 4) for g in (0, 1) if a + g < len(pages)]
            for h in range(Hq):
                kv = h // (Hq // Hkv)
                old = _with_probabilities_in_bf16(f(inp["q_new"][c])[d, h], k[:, kv], v[:, kv], r.shape.scale, pieces)
                err["four pages"] += ((old - ref[d, h]) ** 2).sum()
        err["one piece"] += ((o[c] - ref) ** 2).sum()
    print(err, flush=True)
    assert err["one piece"] <= err["four pages"]


def test_draft_decode_large_logits():
    """Queries twelve times larger: near one-hot rows, reference max far from zero."""
    print("case decode large logits", flush=True)
    inp = make_decode_inputs((700, 90), 5, 16, 2, 64, 1100)
    inp["q_new"] = f32_to_bf16_bits((bf16_bits_to_f64(inp["q_new"]) * 12.0).astype(np.float32))
    r = DecodeRun(inp, 5, 16, 2, 64)
    o, lse, status = r.run()
    assert (status == 0).all()
    _check(inp, o, lse, r.shape.scale, "large logits")


def test_draft_decode_flags_a_block_table_that_points_outside_the_pool():
    """A bad page id or length is caught inside the kernel: the request is flagged, nothing is read out of
    bounds, the other requests are unaffected."""
    print("case decode bad block table", flush=True)
    inp = make_decode_inputs((300, 200, 100), 3, 8, 2, 64, 1110)
    inp["block_table"][1, 2] = inp["n_pages"] + 5           # request 1: page id past the pool
    inp["ctx_len"][2] = 64 * inp["max_pages"] + 1           # request 2: longer than its table can describe
    inp["block_table"][2, :] = inp["block_table"][2, 0]     # (clamped: every block then points at a real page)
    r = DecodeRun(inp, 3, 8, 2, 64)
    o, lse, status = r.run()
    assert status.tolist() == [0, 1, 1]
    ro, rl = _oracle(inp, 0, r.shape.scale)
    assert rel_l2(o[0], ro) <= FWD_REL and max_abs(lse[0], rl) <= LSE_ABS
    assert np.isfinite(lse[1]).all()


def test_draft_decode_replays_from_a_hip_graph():
    """The call allocates nothing and clears nothing with a memset, so a serving loop can capture it: every
    replay (with new queries written between replays) must equal the eager result bit for bit."""
    print("case decode graph replay", flush=True)
    inp = make_decode_inputs((1500, 70, 640), 5, 16, 2, 64, 1120)
    r = DecodeRun(inp, 5, 16, 2, 64)
    r.run()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        pe.peagle_draft_decode(r.shape, r.q, r.k, r.v, r.kp, r.vp, r.bt, r.cl, r.o, r.lse, r.status, r.ws,
                               torch.cuda.current_stream())
    for rep in range(3):
        r.q.copy_(to_dev_bf16(make_decode_inputs((1500, 70, 640), 5, 16, 2, 64, 1130 + rep)["q_new"]))
        r.o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        o_graph, lse_graph = r.o.clone(), r.lse.clone()
        o_eager, lse_eager, _ = r.run()
        assert np.array_equal(bf16_to_f64(o_graph), o_eager), rep
        assert np.array_equal(lse_graph.double().cpu().numpy(), lse_eager), rep


BATCHES = [
    # name, number of requests, largest context, K, Hq, Hkv, D, form (see _form): every kernel, more and fewer workgroups than
    # two per CU, more and fewer pieces than the merge kernels' limits (none, 2, 3 to 8, more)
    ("c64_d64", 64, 2200, 4, 16, 8, 64, (2, True, True)),
    ("c65_d64", 65, 2200, 4, 16, 8, 64, (2, True, False)),
    ("c64_d64_one_piece", 64, 300, 4, 16, 8, 64, (1, True, False)),
    ("c65_d64_one_piece", 65, 300, 4, 16, 8, 64, (1, False, False)),
    ("c64_d128", 64, 2200, 5, 16, 8, 128, (2, False, True)),
    ("c24_d128", 24, 6500, 8, 32, 8, 128, (6, False, True)),
    ("c9_four_row_blocks", 9, 2000, 8, 128, 8, 64, (4, False, False)),
    ("c64_four_row_blocks", 64, 8300, 8, 32, 2, 64, (8, False, True)),
    ("c8_d128", 8, 4096, 3, 32, 8, 128, (4, True, False)),
    ("c2_d128_many_pieces", 2, 20000, 5, 32, 4, 128, (32, True, False)),
    ("c4_d128_one_piece", 4, 500, 5, 32, 4, 128, (1, True, False)),
    ("c70_d128_one_piece_three_row_blocks", 70, 500, 6, 64, 4, 128, (1, False, False)),
    ("c9_d128_three_row_blocks", 9, 4096, 5, 64, 4, 128, (7, False, False)),
]


@pytest.mark.parametrize("name,C,longest,K,Hq,Hkv,D,form", BATCHES, ids=[c[0] for c in BATCHES])
def test_draft_decode_batches(name, C, longest, K, Hq, Hkv, D, form):
    """Lengths with ties, empty requests and the longest anywhere; then one request's table is spoiled: it alone is
    flagged and no other request's output changes."""
    rng = np.random.default_rng(C + D)
    lens = rng.integers(0, longest, C)
    lens[rng.integers(0, C, 4)] = 64
    lens[rng.integers(0, C, 3)] = 0
    lens[C // 2] = longest
    print(f"case decode {name}: ctx={lens.tolist()} K={K} Hq={Hq} Hkv={Hkv} D={D}", flush=True)
    inp = make_decode_inputs(tuple(int(x) for x in lens), K, Hq, Hkv, D, 1100 + C)
    r = DecodeRun(inp, K, Hq, Hkv, D)
    assert _form(r.shape) == form
    o, lse, status = r.run()
    assert (status == 0).all()
    _check(inp, o, lse, r.shape.scale, name)
    r.bt[C // 2, 0] = r.shape.n_pages                        # outside the pool: skipped and flagged
    o2, lse2, status2 = r.run()
    others = np.arange(C) != C // 2
    assert status2[C // 2] == 1 and (status2[others] == 0).all()
    assert np.array_equal(o2[others], o[others]) and np.array_equal(lse2[others], lse[others])


@pytest.mark.parametrize("longest", [1000, 2 * 16 * 64, 2 * 16 * 64 + 1, 8192])
def test_draft_decode_in_a_table_wider_than_its_requests(longest):
    """Sixty-four requests in a table of 128 pages, two pieces each: taken by falling length only if one of them is longer
    than two pieces of sixteen pages."""
    C, K, Hq, Hkv, D = 64, 4, 16, 8, 64
    rng = np.random.default_rng(longest)
    lens = rng.integers(0, 1000, C)
    lens[C // 3] = longest
    print(f"case decode wide table: longest {longest}", flush=True)
    inp = make_decode_inputs(tuple(int(x) for x in lens), K, Hq, Hkv, D, 1200)
    table = np.full((C, 128), -1, dtype=np.int32)
    table[:, :inp["max_pages"]] = inp["block_table"]
    r = DecodeRun(inp | {"block_table": table, "max_pages": 128}, K, Hq, Hkv, D)
    assert pe.peagle_draft_decode_splits(r.shape) == 2
    o, lse, status = r.run()
    assert (status == 0).all()
    _check(inp, o, lse, r.shape.scale, f"wide table {longest}")


@pytest.mark.parametrize("C,ctx,Hq,Hkv,D", [(4, 4096, 64, 8, 64), (1, 20000, 8, 8, 64), (55, 2469, 64, 8, 64), (3, 700, 16, 2, 64),
                                             (16, 8192, 32, 4, 128), (35, 3838, 32, 4, 128), (5, 512, 32, 4, 128)])
def test_draft_decode_leaves_a_partial_record_for_each_piece(C, ctx, Hq, Hkv, D):
    """peagle_draft_decode_splits() pieces of every request and KV head each leave one record of unnormalised rows at the
    start of the workspace; a single piece leaves none."""
    print(f"case decode records: {C} of {ctx} Hq={Hq} Hkv={Hkv} D={D}", flush=True)
    K, pages = 3, -(-ctx // 64)
    shape = pe.DecodeShape(C, K, Hq, Hkv, D, 8, pages)
    rows_pad = -(-K * (Hq // Hkv) // 32) * 32
    rec = rows_pad * D
    g = torch.Generator(device="cuda").manual_seed(1400 + C)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v, kp, vp = rnd(C, K, Hq, D), rnd(C, K, Hkv, D), rnd(C, K, Hkv, D), rnd(8, Hkv, 64, D), rnd(8, Hkv, 64, D)
    table = torch.randint(0, 8, (C, pages), generator=g, device="cuda", dtype=torch.int32)
    lens, status = (torch.full((C,), n, dtype=torch.int32, device="cuda") for n in (ctx, -7))
    o, lse = torch.empty_like(q), torch.empty((C, Hq, K), device="cuda")
    ws = torch.full((pe.peagle_draft_decode_workspace_bytes(shape),), 0x5A, dtype=torch.uint8, device="cuda")
    pe.peagle_draft_decode(shape, q, k, v, kp, vp, table, lens, o, lse, status, ws)
    torch.cuda.synchronize()
    assert (status == 0).all()
    laid_out = ws.numel() // (4 * rows_pad * (D + 3))        # (beside a record's rows: maximum, sum and flag of each)
    written = (ws[:4 * laid_out * rec].view(torch.int32).view(laid_out, rec) != 0x5A5A5A5A).any(1).cpu().numpy()
    pieces = pe.peagle_draft_decode_splits(shape)
    assert written.tolist() == [pieces > 1 and r < C * Hkv * pieces for r in range(laid_out)]


@pytest.mark.parametrize("D,pages", [(64, 1), (64, 12), (64, 13), (128, 8), (128, 9)])
def test_draft_decode_with_one_piece_and_with_more(D, pages):
    """Tables of up to 12 (D = 64) or 8 (D = 128) pages are not cut: the kernel leaves output, LSE and status itself.  Two
    blocks of 32 query rows, the second ragged; empty, page-edge and full requests; one with a page outside the pool."""
    K, Hq, Hkv, n = 5, 16, 2, 64 * pages
    lens = (n, 0, 1, n - 1, min(n, 65), n, 64)
    print(f"case decode one piece: {pages} pages D={D}", flush=True)
    inp = make_decode_inputs(lens, K, Hq, Hkv, D, 1300 + pages)
    r = DecodeRun(inp, K, Hq, Hkv, D)
    assert r.shape.max_pages == pages
    o, lse, status = r.run()
    assert (status == 0).all()
    _check(inp, o, lse, r.shape.scale, f"one piece {pages} {D}")
    r.bt[5, pages - 1] = r.shape.n_pages
    o2, lse2, status2 = r.run()
    assert status2.tolist() == [0, 0, 0, 0, 0, 1, 0]
    others = np.arange(len(lens)) != 5
    assert np.array_equal(o2[others], o[others]) and np.array_equal(lse2[others], lse[others])


@pytest.mark.parametrize("K,Hq,Hkv", [(1, 3, 3), (3, 5, 1), (5, 21, 3), (16, 8, 1), (42, 9, 3)])
@pytest.mark.parametrize("D,ctx,at_least", [(64, 800, 2), (64, 1500, 3), (64, 4000, 9), (128, 600, 2), (128, 1200, 3), (128, 4000, 9)])
def test_draft_decode_merges_pieces_of_any_number_of_rows(D, ctx, at_least, K, Hq, Hkv):
    """One, 15, 35, 128 (the most) and 126 rows per KV head, none a whole number of the merging workgroups' rows but
    the fourth; two to sixteen pieces, so that each form of the merging kernel runs; one request with a bad page."""
    print(f"case decode merge ctx={ctx} K={K} Hq={Hq} Hkv={Hkv} D={D}", flush=True)
    inp = make_decode_inputs((ctx, ctx // 3), K, Hq, Hkv, D, 1600 + K)
    r = DecodeRun(inp, K, Hq, Hkv, D)
    assert pe.peagle_draft_decode_splits(r.shape) >= at_least
    o, lse, status = r.run()
    assert (status == 0).all()
    _check(inp, o, lse, r.shape.scale, f"merge {ctx} {K}")
    r.bt[1, 1] = r.shape.n_pages
    assert r.run()[2].tolist() == [0, 1]


def test_draft_decode_refuses_more_than_128_rows_per_kv_head():
    assert pe.peagle_draft_decode_workspace_bytes(pe.DecodeShape(2, 42, 9, 3, 64, 8, 8)) > 0
    with pytest.raises(pe.PeagleError):
        pe.peagle_draft_decode_workspace_bytes(pe.DecodeShape(2, 43, 9, 3, 64, 8, 8))
