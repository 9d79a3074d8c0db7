"""GPU parity tests: the HIP path (through the C ABI) against the fp64 oracle on the same seeded
inputs.  Tolerances are the ones fixed for this path: tile map bit-exact (host tests), forward
max-abs <= 1e-2 and rel-L2 <= 5e-3, gradients rel-L2 <= 1e-2, partitioned vs unpartitioned
rel-L2 <= 1e-3.  Every case prints what it is before touching the GPU."""
import numpy as np
import pytest
import torch

import paper_2602_01469_amd as pe
from gpu_harness import Run, bf16_to_f64, dq_path, fwd_form, max_abs, mean_list, one_head_per_cu, rand_bits, rel_l2, to_dev_bf16
from oracle import peagle_oracle as orc
from peagle_inputs import CONFIGS, bf16_bits_to_f64, make_inputs

pytestmark = pytest.mark.gpu

FWD_MAX_ABS, FWD_REL, GRAD_REL, PART_REL = 1e-2, 5e-3, 1e-2, 1e-3
# LSE = m + log(sum of the bf16-rounded probabilities that also enter P V): the sum carries the
# bf16 rounding of its terms (8-bit significand: at most 2^-8 relative), i.e. 2^-8 in the logarithm.
LSE_ABS = 4e-3


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# Share of O elements that may exceed 1e-2 (only where the bf16 formats force it, see _check_o_abs): such
# elements need |O| >= 2, i.e. a row that puts nearly all its weight on one key whose |V| is at least 2.
O_OVER_CAP = 2e-5


def _bf16_half_ulp(x):
    """Half the spacing of bf16 numbers (8-bit significand) at |x|."""
    return 2.0 ** (np.floor(np.log2(np.maximum(np.abs(x), 2.0 ** -126))) - 8)


def _check_o_abs(o, ref, what, extra=0.0):
    """|O - ref| <= 1e-2 for every element the bf16 formats allow it for, i.e. wherever |ref| < 2.

    O is stored in bf16 and the probabilities enter P V in bf16 (the path's stated arithmetic): an element
    carries up to half an output ulp plus, when the row's weight sits on few keys, up to 2^-9 |O| from the
    rounding of those probabilities.  Below |O| = 2 that is at most 2^-8 + 2^-8 = 7.8e-3, inside the fixed
    bound, which is then applied as it stands.  From |O| = 2 on the two terms alone reach 1.2e-2, so there the
    bound is half an output ulp + 2^-9 |O| + 2e-3 for everything else; the count of elements above 1e-2 is
    printed and capped.  ``extra`` widens every bound by a stated, derived amount (operand rounding that the
    reference does not share: the rotary tests)."""
    err = np.abs(o - ref)
    forced = _bf16_half_ulp(ref) + np.abs(ref) * 2.0 ** -9 + 2e-3
    bound = np.where(np.abs(ref) < 2.0, FWD_MAX_ABS, np.maximum(FWD_MAX_ABS, forced)) + extra
    bad = err > bound
    if bad.any():
        w = np.unravel_index(np.argmax(err - bound), err.shape)
        raise AssertionError(f"{what}: {int(bad.sum())} O elements over the bound; worst at {w}: got {o[w]!r} "
                             f"ref {ref[w]!r} err {err[w]:.3e} bound {bound[w]:.3e}; max err {err.max():.3e}")
    over = int((err > FWD_MAX_ABS + extra).sum())
    print(f"{what}: O max abs err {err.max():.3e} (over 1e-2: {over} of {err.size}, all at |O| >= 2)", flush=True)
    assert over <= max(1, int(O_OVER_CAP * err.size)), (what, over, err.size)


def _check_against_oracle(got, ref, what="", lse_abs=LSE_ABS, o_abs_extra=0.0):
    assert not any(np.isnan(got[n]).any() for n in got), what
    assert rel_l2(got["O"], ref["O"]) <= FWD_REL, what
    _check_o_abs(got["O"], ref["O"], what, o_abs_extra)
    assert max_abs(got["LSE"], ref["LSE"]) <= lse_abs, what
    for n in ("dQ", "dK", "dV"):
        assert _grad_rel(got[n], ref[n]) <= GRAD_REL, (what, n)


def _grad_rel(got, ref):
    """rel-L2 of a gradient, the reference norm floored at an rms of 1e-3 (unit-variance inputs give gradients
    with an rms of 0.1 to 1): a problem whose rows all see a single key (one anchor, K = 1) has dQ = 0 exactly,
    where the kernel's dP - Delta leaves rounding noise of 1e-7 and a plain ratio is meaningless."""
    return float(np.linalg.norm((got - ref).ravel()) / max(np.linalg.norm(ref.ravel()), 1e-3 * np.sqrt(ref.size)))


def _oracle(qb, kb, vb, dob, L, K, scale):
    q, k, v, do = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    return orc.attn_backward(q, k, v, do, L, K, scale)


SMALL = [
    # name, L, K, Hq, Hkv, D, seed, bounds, L_max
    ("even_group", 128, 4, 4, 1, 64, 100, None, None),
    ("odd_group", 128, 4, 3, 3, 64, 110, None, None),
    ("ragged_tail", 100, 8, 4, 2, 64, 120, None, None),
    ("k_not_dividing_128", 50, 3, 2, 1, 64, 130, None, None),
    ("k1_plain_causal", 300, 1, 2, 2, 64, 140, None, None),
    ("single_anchor", 1, 8, 2, 1, 64, 150, None, None),
    ("k16", 40, 16, 2, 2, 64, 160, None, None),
    ("segments", 256, 8, 4, 2, 64, 170, [0, 64, 128, 256], None),
    ("segments_cropped", 219, 8, 4, 2, 64, 180, [0, 64, 128, 256], 256),
    ("crop_to_one_segment", 60, 8, 4, 2, 64, 190, [0, 64, 128, 256], 256),
    ("d128", 128, 4, 4, 2, 128, 200, None, None),
    ("d128_one_head", 96, 8, 1, 1, 128, 210, None, None),
    ("d128_segments_cropped", 200, 8, 2, 1, 128, 220, [0, 64, 128, 256], 256),
    ("several_tiles", 700, 4, 4, 2, 64, 230, [0, 256, 512, 700], None),
    ("group_of_12", 150, 8, 12, 1, 64, 240, [0, 64, 150], None),
    ("seven_mha_heads", 90, 4, 7, 7, 64, 250, None, None),
    ("odd_group_d128", 70, 8, 9, 3, 128, 260, None, None),
    # deep chains up to the largest supported K (one anchor per row tile), and depths that do not divide 128
    ("k32", 20, 32, 2, 1, 64, 270, None, None),
    ("k64_segments", 9, 64, 2, 2, 64, 280, [0, 4, 9], None),
    ("k128_largest_depth", 5, 128, 2, 1, 64, 290, [0, 2, 5], None),
    ("k128_d128", 3, 128, 1, 1, 128, 293, None, None),
    ("k5_segments", 60, 5, 4, 2, 64, 291, [0, 25, 60], None),
    ("k7_d128", 40, 7, 2, 1, 128, 292, None, None),
    ("k2", 200, 2, 2, 1, 64, 294, [0, 64, 200], None),
]


@pytest.mark.parametrize("name,L,K,Hq,Hkv,D,seed,bounds,L_max", SMALL, ids=[c[0] for c in SMALL])
def test_small_cases_match_oracle(name, L, K, Hq, Hkv, D, seed, bounds, L_max):
    print(f"case {name}: L={L} K={K} Hq={Hq} Hkv={Hkv} D={D} seed={seed} bounds={bounds} L_max={L_max}", flush=True)
    T = L * K
    qb, kb, vb, dob = (rand_bits((T, Hq, D), seed), rand_bits((T, Hkv, D), seed + 1), rand_bits((T, Hkv, D), seed + 2),
                       rand_bits((T, Hq, D), seed + 3))
    tm = pe.peagle_build_tilemap(L_max or L, K, bounds, device=0)
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.fwd()
    r.bwd()
    got = r.results()
    ref = _oracle(qb, kb, vb, dob, L, K, r.shape.scale)
    _check_against_oracle(got, ref, name)
    if bounds is not None:
        S = len(bounds) - 1
        r2 = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        dkb = torch.empty((T, Hkv, D), dtype=torch.bfloat16, device="cuda")
        dvb = torch.empty((T, Hkv, D), dtype=torch.bfloat16, device="cuda")
        r2.step(0, S, dkb, dvb)
        g2 = r2.results()
        _check_against_oracle(g2, ref, name + " partitioned")
        for n in ("O", "LSE", "dQ"):
            assert np.array_equal(g2[n], got[n]), n      # a row is computed by exactly one segment, identically
        for n in ("dK", "dV"):
            assert rel_l2(g2[n], got[n]) <= PART_REL, n
        assert np.array_equal(bf16_to_f64(dkb), bf16_to_f64(r2.dk.to(torch.bfloat16)))
        assert np.array_equal(bf16_to_f64(dvb), bf16_to_f64(r2.dv.to(torch.bfloat16)))
        # resumed run: segments [0,1) then [1,S) on the same accumulators
        r3 = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r3.step(0, 1)
        r3.step(1, S)
        g3 = r3.results()
        for n in ("O", "LSE", "dQ", "dK", "dV"):
            assert np.array_equal(g3[n], g2[n]), n
        # per-segment backward with explicit accumulation into zeroed buffers
        r4 = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r4.dk.zero_()
        r4.dv.zero_()
        for s in range(S):
            r4.fwd(s)
            r4.bwd(s, accumulate=1)
        g4 = r4.results()
        for n in ("dK", "dV"):
            assert rel_l2(g4[n], got[n]) <= PART_REL, n


@pytest.mark.parametrize("bounds", [None, [0, 1040, 1500]], ids=["one_pass", "two_segments"])
def test_dense_segments_of_many_row_tiles(bounds):
    """94 row tiles in one segment (or 65 + 29): more row tiles than key-tile pairs in one dK/dV launch, and a second
    segment adding to what the first wrote, each followed by its own reduction; every element of every output
    against the oracle.  (Segments cut into several launches: test_dense_segments_of_more_than_128_row_tiles.)"""
    L, K, Hq, Hkv, D, seed = 1500, 8, 2, 1, 64, 290
    print(f"case dense long segments: L={L} K={K} Hq={Hq} Hkv={Hkv} D={D} seed={seed} bounds={bounds}", flush=True)
    qb, kb, vb, dob = (rand_bits((L * K, H, D), seed + i) for i, H in enumerate((Hq, Hkv, Hkv, Hq)))
    tm = pe.peagle_build_tilemap(L, K, bounds, device=0)
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.step(0, 1 if bounds is None else len(bounds) - 1)
    got = r.results()
    ref = _oracle(qb, kb, vb, dob, L, K, r.shape.scale)
    _check_against_oracle(got, ref, f"dense long segments {bounds}")
    for n in ("dK", "dV"):                      # no key left out or counted twice at a launch boundary
        assert max_abs(got[n], ref[n]) <= 2e-2 * np.abs(ref[n]).max(), n
    r.fwd()                                     # the single-segment entry points take the same path
    r.bwd()
    whole = r.results()
    for n in ("O", "LSE", "dQ"):
        assert np.array_equal(whole[n], got[n]), n
    for n in ("dK", "dV"):
        assert rel_l2(got[n], whole[n]) <= PART_REL, n


@pytest.mark.parametrize("Hq,Hkv", [(56, 14), (56, 28)])
def test_two_heads_per_forward_workgroup_match_oracle(Hq, Hkv):
    """Lists long enough (mean above 10) and heads enough for the forward to take the heads of a group two at a time at D =
    64, three workgroups per CU; the first and the last KV head's groups against the oracle."""
    L, K, D, seed = 1290, 4, 64, 296
    print(f"case two heads per workgroup Hq={Hq} Hkv={Hkv}", flush=True)
    qb, kb, vb, dob = (rand_bits((L * K, H, D), seed + i) for i, H in enumerate((Hq, Hkv, Hkv, Hq)))
    tm = pe.peagle_build_tilemap(L, K, [0, 640, L], device=0)
    assert fwd_form(tm, Hq, Hkv) == "two heads, three per CU"
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.step(0, 2)
    got = r.results()
    for h in (0, Hkv - 1):
        a, b = slice(h * (Hq // Hkv), (h + 1) * (Hq // Hkv)), slice(h, h + 1)
        part = {"O": got["O"][:, a], "LSE": got["LSE"][a], "dQ": got["dQ"][:, a], "dK": got["dK"][:, b], "dV": got["dV"][:, b]}
        _check_against_oracle(part, _oracle(qb[:, a], kb[:, b], vb[:, b], dob[:, a], L, K, r.shape.scale), f"two heads, group {h}")


@pytest.mark.parametrize("L,Hq", [(600, 4), (2000, 4), (2000, 52)])
@pytest.mark.parametrize("qscale", [10.0, 12.0, 40.0])
def test_large_logits_take_the_running_max_path(qscale, L, Hq):
    """Scores far outside the exponent range that the forward's first pass (reference max fixed at
    0) can hold: the kernel must detect it and redo the row tile with the running-max form, with one head
    per workgroup and (52 heads) with two.  The dQ kernel leaves its probabilities unnormalised only
    while |lse| <= 64 in log2 units: at the smaller scales some workgroups are inside that range and some
    outside, at the largest none is inside.  Both sequences are long enough for the pipelined kernel's
    groups of three full tiles to occur in the one grid; 52 heads take the plain kernel.  The first two KV heads against the
    oracle."""
    K, Hkv, D = 4, Hq // 2, 64
    print(f"case large_logits qscale={qscale} L={L} Hq={Hq}", flush=True)
    T = L * K
    qb, kb, vb, dob = (rand_bits((T, Hq, D), 300, qscale), rand_bits((T, Hkv, D), 301), rand_bits((T, Hkv, D), 302),
                       rand_bits((T, Hq, D), 303))
    tm = pe.peagle_build_tilemap(L, K, None, device=0)
    assert fwd_form(tm, Hq, Hkv) == ("one head" if Hq == 4 else "two heads, three per CU")
    assert (mean_list(tm) < 10) == (L == 600) and (mean_list(tm) > 11) == (L == 2000)
    assert dq_path(tm, Hq, "backward") == ("plain" if Hq == 52 else "one grid")
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.fwd()
    r.bwd()
    got = r.results()
    assert not any(np.isnan(got[n]).any() for n in got)
    got = {"O": got["O"][:, :4], "LSE": got["LSE"][:4], "dQ": got["dQ"][:, :4], "dK": got["dK"][:, :2], "dV": got["dV"][:, :2]}
    ref = _oracle(qb[:, :4], kb[:, :2], vb[:, :2], dob[:, :4], L, K, r.shape.scale)
    outside = np.abs(ref["LSE"]) * np.log2(np.e) > 64                                  # [Hq, K * L]
    row_tile = np.arange(T) % L // 32
    share = np.mean([outside[h, row_tile == t].any() for h in range(4) for t in range(row_tile.max() + 1)])
    assert share == 1 if qscale == 40.0 else 0 < share < 1, share                      # workgroups outside dQ's range
    lse_span = ref["LSE"].max() - ref["LSE"].min()
    assert lse_span > 60 * (qscale / 12.0)       # the case really leaves the comfortable range
    assert rel_l2(got["O"], ref["O"]) <= FWD_REL
    # |LSE| is in the hundreds here: fp32 resolution of the stored value dominates the bf16-sum term
    assert max_abs(got["LSE"], ref["LSE"]) <= LSE_ABS + 2e-6 * np.abs(ref["LSE"]).max()
    for n in ("dQ", "dK", "dV"):
        assert rel_l2(got[n], ref[n]) <= GRAD_REL, n


def _heads_run(tm, L, K, q, k, v, d_o, profiled=False):
    """A step (profiled: its kernels launched apart) over the heads given, [T, H, D] tensors on the device."""
    shape = pe.Shape(L, K, q.shape[1], k.shape[1], q.shape[2])
    o, dq = (torch.full_like(q, float("nan")) for _ in range(2))
    lse = torch.full((q.shape[1], q.shape[0]), float("nan"), device="cuda")
    dk, dv = (torch.full(k.shape, float("nan"), device="cuda") for _ in range(2))
    ws = torch.empty(pe.peagle_workspace_bytes(tm, shape), dtype=torch.uint8, device="cuda")
    if profiled:
        pe.peagle_attn_step_profiled(tm, shape, 0, tm.info()["S"], q, k, v, d_o, o, lse, dq, dk, dv, ws)
    else:
        pe.peagle_attn_step_partitioned(tm, shape, 0, tm.info()["S"], q, k, v, d_o, o, lse, dq, dk, dv, None, None, ws)
    torch.cuda.synchronize()
    return {"o": o, "dq": dq, "lse": lse.t(), "dk": dk, "dv": dv}


@pytest.mark.parametrize("D", [64, 128])
def test_a_head_does_not_depend_on_the_heads_beside_it(D):
    """Heads of ordinary and of very large logits in turn.  At D = 64 two heads of a group share a forward workgroup where
    heads are many and lists long, none where they are not: heads alone, and the crop to short lists, give the same bits."""
    L, K, Hq, Hkv, Lc = 2000, 4, 36, 18, 896
    print(f"case neighbouring heads D={D}", flush=True)
    tm = pe.peagle_build_tilemap(L, K, None, device=0)
    assert fwd_form(tm, Hq, Hkv) == "two heads, three per CU" and fwd_form(tm, 1, 1) == "one head"
    assert fwd_form(pe.peagle_build_tilemap(Lc, K, None, device=-1), Hq, Hkv) == "one head"
    g = torch.Generator(device="cuda").manual_seed(340)
    q, k, v, d_o = (torch.randn(L * K, H, D, generator=g, device="cuda") for H in (Hq, Hkv, Hkv, Hq))
    q[:, 1::2] *= 40.0
    q, k, v, d_o = (t.to(torch.bfloat16) for t in (q, k, v, d_o))
    whole = _heads_run(tm, L, K, q, k, v, d_o)
    for h in (0, 1, 2, 17, Hq - 2, Hq - 1):
        b = slice(h // 2, h // 2 + 1)
        alone = _heads_run(tm, L, K, q[:, h:h + 1].contiguous(), k[:, b].contiguous(), v[:, b].contiguous(),
                           d_o[:, h:h + 1].contiguous())
        for n in ("o", "lse", "dq"):
            assert torch.equal(whole[n][:, h:h + 1], alone[n]), (n, h)
    cut = lambda t: t.reshape(K, L, t.shape[1], -1)[:, :Lc].reshape(K * Lc, t.shape[1], -1).contiguous()
    crop = _heads_run(tm, Lc, K, *(cut(t) for t in (q, k, v, d_o)))
    for n in ("o", "lse", "dq"):                    # (896 anchors are whole row tiles)
        assert torch.equal(cut(whole[n]).view_as(crop[n]), crop[n]), n


@pytest.mark.parametrize("Hq,Hkv", [(8, 4), (16, 4)], ids=["two_per_cu", "three_per_cu"])
def test_two_head_forward_workgroups_give_the_bits_of_one_head_ones(Hq, Hkv):
    """752 and 1,504 workgroups of two heads with long lists (the forward's two-head forms at D = 64) against each group of
    heads alone (few workgroups: one head each); every other head's row tiles are done again with the running max."""
    L, K, D = 3000, 8, 64
    print(f"case forward forms Hq={Hq}", flush=True)
    tm = pe.peagle_build_tilemap(L, K, None, device=0)
    assert fwd_form(tm, Hq, Hkv) == ("two heads, two per CU" if Hq == 8 else "two heads, three per CU")
    assert fwd_form(tm, Hq // Hkv, 1) == "one head"
    g = torch.Generator(device="cuda").manual_seed(341)
    q, k, v, d_o = (torch.randn(L * K, H, D, generator=g, device="cuda") for H in (Hq, Hkv, Hkv, Hq))
    q[:, 1::2] *= 40.0
    q, k, v, d_o = (t.to(torch.bfloat16) for t in (q, k, v, d_o))
    whole = _heads_run(tm, L, K, q, k, v, d_o)
    n = Hq // Hkv
    for h in range(Hkv):
        a, b = slice(h * n, (h + 1) * n), slice(h, h + 1)
        alone = _heads_run(tm, L, K, *(t.contiguous() for t in (q[:, a], k[:, b], v[:, b], d_o[:, a])))
        for name in ("o", "lse"):
            assert torch.isfinite(alone[name]).all(), name
            assert torch.equal(whole[name][:, a], alone[name]), (name, h)


def test_run_to_run_determinism():
    L, K, Hq, Hkv, D = 300, 8, 4, 2, 64
    print("case determinism", flush=True)
    T = L * K
    qb, kb, vb, dob = (rand_bits((T, Hq, D), 1), rand_bits((T, Hkv, D), 2), rand_bits((T, Hkv, D), 3),
                       rand_bits((T, Hq, D), 4))
    tm = pe.peagle_build_tilemap(L, K, None, device=0)
    outs = []
    for _ in range(2):
        r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r.fwd()
        r.bwd()
        outs.append(r.results())
    for n in outs[0]:
        assert np.array_equal(outs[0][n], outs[1][n]), n


def test_zero_query_closed_form_on_gpu():
    """Q == 0 gives uniform attention: O is the mean of the visible V rows and LSE = ln(i+1+d)."""
    L, K, Hq, Hkv, D = 200, 4, 2, 1, 64
    print("case zero_query", flush=True)
    T = L * K
    qb = np.zeros((T, Hq, D), dtype=np.uint16)
    kb, vb, dob = rand_bits((T, Hkv, D), 5), rand_bits((T, Hkv, D), 6), rand_bits((T, Hq, D), 7)
    tm = pe.peagle_build_tilemap(L, K, None, device=0)
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.fwd()
    got = r.results()
    v = bf16_bits_to_f64(vb)[:, 0]
    i, d = np.arange(T) % L, np.arange(T) // L
    assert np.abs(got["LSE"] - np.log(i + 1 + d)[None, :]).max() < 1e-5   # every p is exactly 1
    csum = np.cumsum(v[:L], axis=0)
    for t in range(0, T, 37):
        mean = (csum[i[t]] + sum(v[e * L + i[t]] for e in range(1, d[t] + 1))) / (i[t] + 1 + d[t])
        assert np.abs(got["O"][t, 0] - mean).max() < 1e-2


def test_c1_tiny_config():
    cfg = CONFIGS["c1_tiny"]
    print(f"case {cfg.name}", flush=True)
    qb, kb, vb, dob = make_inputs(cfg)
    tm = pe.peagle_build_tilemap(cfg.L, cfg.K, cfg.seg_bounds(), device=0)
    r = Run(tm, cfg.L, cfg.K, cfg.Hq, cfg.Hkv, cfg.D, qb, kb, vb, dob, cfg.scale)
    r.step(0, 1)
    _check_against_oracle(r.results(), _oracle(qb, kb, vb, dob, cfg.L, cfg.K, cfg.scale), cfg.name)


def test_c2_gptoss_one_whole_kv_group():
    """Full-size config 2; the oracle covers one complete KV group (all its 8 query heads, all rows)."""
    cfg = CONFIGS["c2_gptoss"]
    print(f"case {cfg.name}", flush=True)
    qb, kb, vb, dob = make_inputs(cfg)
    tm = pe.peagle_build_tilemap(cfg.L, cfg.K, cfg.seg_bounds(), device=0)
    r = Run(tm, cfg.L, cfg.K, cfg.Hq, cfg.Hkv, cfg.D, qb, kb, vb, dob, cfg.scale)
    r.step(0, 1)
    got = r.results()
    g = 5
    grp = cfg.Hq // cfg.Hkv
    hs = slice(g * grp, (g + 1) * grp)
    ref = _oracle(qb[:, hs], kb[:, g:g + 1], vb[:, g:g + 1], dob[:, hs], cfg.L, cfg.K, cfg.scale)
    sub = {"O": got["O"][:, hs], "LSE": got["LSE"][hs], "dQ": got["dQ"][:, hs], "dK": got["dK"][:, g:g + 1],
           "dV": got["dV"][:, g:g + 1]}
    _check_against_oracle(sub, ref, cfg.name)
    _check_global_identities(got, qb, kb, dob, cfg)


def _check_global_identities(got, qb, kb, dob, cfg):
    """Properties that hold at any size: softmax rows sum to one, so sum_keys dV = sum_rows dO per KV
    head; the score gradient seen from the query and the key side agrees: sum dQ.Q = sum dK.K."""
    grp = cfg.Hq // cfg.Hkv
    do = bf16_bits_to_f64(dob)
    lhs = got["dV"].sum(axis=0)                                              # [Hkv, D]
    rhs = do.sum(axis=0).reshape(cfg.Hkv, grp, cfg.D).sum(axis=1)
    assert np.abs(lhs - rhs).max() <= 2e-3 * np.abs(do).sum(axis=0).reshape(cfg.Hkv, grp, cfg.D).sum(axis=1).max()
    q = bf16_bits_to_f64(qb)
    k = bf16_bits_to_f64(kb)
    a = (got["dQ"] * q).sum(axis=(0, 2)).reshape(cfg.Hkv, grp).sum(axis=1)
    b = (got["dK"] * k).sum(axis=(0, 2))
    scale_ref = np.sqrt((got["dQ"] ** 2).sum() * (q ** 2).sum() / cfg.Hkv)
    assert np.abs(a - b).max() <= 1e-3 * scale_ref


def _sampled_check(cfg, got, qb, kb, vb, dob, g, n_anchor_samples=6, seed=0):
    """Oracle on sampled query rows (every depth of sampled anchors) for one KV group: O, LSE, dQ of
    those rows; and dK/dV of the last anchors' keys, whose visible rows (all rows of those anchors)
    the oracle computes in full."""
    L, K = cfg.L, cfg.K
    grp = cfg.Hq // cfg.Hkv
    hs = slice(g * grp, (g + 1) * grp)
    q, k, v, do = (bf16_bits_to_f64(x) for x in (qb[:, hs], kb[:, g:g + 1], vb[:, g:g + 1], dob[:, hs]))
    rng = np.random.default_rng(seed)
    anchors = np.unique(np.concatenate([[0, 1, 63, 64, L // 2, L - 1], rng.integers(0, L, size=n_anchor_samples)]))
    rows = np.concatenate([d * L + anchors for d in range(K)])
    ref = orc.attn_backward(q, k, v, do, L, K, cfg.scale, rows=rows, row_block=256)
    assert rel_l2(got["O"][rows][:, hs], ref["O"]) <= FWD_REL
    _check_o_abs(got["O"][rows][:, hs], ref["O"], cfg.name if hasattr(cfg, "name") else "sampled")
    assert max_abs(got["LSE"][hs][:, rows], ref["LSE"]) <= LSE_ABS
    assert rel_l2(got["dQ"][rows][:, hs], ref["dQ"]) <= GRAD_REL
    # keys of the last `tail` anchors are seen only by rows of those anchors
    tail = 40
    a0 = L - tail
    rows2 = np.concatenate([d * L + np.arange(a0, L) for d in range(K)])
    ref2 = orc.attn_backward(q, k, v, do, L, K, cfg.scale, rows=rows2, row_block=256)
    for n in ("dK", "dV"):
        assert rel_l2(got[n][rows2][:, g:g + 1], ref2[n][rows2]) <= GRAD_REL, n


def _prefix_inputs(bits_list, L, Lp, K):
    idx = np.concatenate([d * L + np.arange(Lp) for d in range(K)])
    return [np.ascontiguousarray(b[idx]) for b in bits_list], idx


@pytest.mark.parametrize("name", ["c3_median", "c4_p90"])
def test_full_size_partitioned_configs(name):
    """Configs 3 and 4 in the launch configuration the benchmark times (partitioned step)."""
    cfg = CONFIGS[name]
    print(f"case {name}: generating inputs", flush=True)
    qb, kb, vb, dob = make_inputs(cfg)
    b = cfg.seg_bounds()
    tm = pe.peagle_build_tilemap(cfg.L, cfg.K, b, device=0)
    r = Run(tm, cfg.L, cfg.K, cfg.Hq, cfg.Hkv, cfg.D, qb, kb, vb, dob, cfg.scale)
    print(f"case {name}: partitioned step, {len(b) - 1} segments", flush=True)
    r.step(0, len(b) - 1)
    got = r.results()
    assert not any(np.isnan(got[n]).any() for n in got)
    print(f"case {name}: oracle on sampled rows", flush=True)
    _sampled_check(cfg, got, qb, kb, vb, dob, g=cfg.Hkv - 1)
    _check_global_identities(got, qb, kb, dob, cfg)
    print(f"case {name}: unpartitioned run", flush=True)
    r.fwd()
    r.bwd()
    whole = r.results()
    for n in ("O", "LSE", "dQ"):
        assert np.array_equal(whole[n], got[n]), n
    for n in ("dK", "dV"):
        assert rel_l2(got[n], whole[n]) <= PART_REL, n


def test_c3_median_one_whole_kv_group_all_rows():
    """Config 3 as the benchmark runs it (4 segments), the oracle on one complete KV group - its 8 query heads,
    all 32,768 rows - so that O, LSE, dQ of every row and dK, dV of every key of the group are compared.  The
    oracle runs segment by segment as well (its own partitioned form, which holds a segment's rows and keys)."""
    cfg = CONFIGS["c3_median"]
    print(f"case {cfg.name}: whole KV group, generating inputs", flush=True)
    qb, kb, vb, dob = make_inputs(cfg)
    b = cfg.seg_bounds()
    tm = pe.peagle_build_tilemap(cfg.L, cfg.K, b, device=0)
    r = Run(tm, cfg.L, cfg.K, cfg.Hq, cfg.Hkv, cfg.D, qb, kb, vb, dob, cfg.scale)
    r.step(0, len(b) - 1)
    got = r.results()
    g = 2
    grp = cfg.Hq // cfg.Hkv
    hs = slice(g * grp, (g + 1) * grp)
    print(f"case {cfg.name}: oracle on KV head {g} (query heads {g * grp}..{(g + 1) * grp - 1}), all rows", flush=True)
    q, k, v, do = (bf16_bits_to_f64(x) for x in (qb[:, hs], kb[:, g:g + 1], vb[:, g:g + 1], dob[:, hs]))
    ref = orc.attn_step_partitioned(q, k, v, do, cfg.L, cfg.K, cfg.scale, b, row_block=2048)
    sub = {"O": got["O"][:, hs], "LSE": got["LSE"][hs], "dQ": got["dQ"][:, hs], "dK": got["dK"][:, g:g + 1],
           "dV": got["dV"][:, g:g + 1]}
    _check_against_oracle(sub, ref, cfg.name + " whole group")
    for n in ("dK", "dV"):
        assert max_abs(sub[n], ref[n]) <= 2e-2 * np.abs(ref[n]).max(), n


def test_c5_p99_stress_prefix_and_samples():
    """Config 5: partitioned run at L=20480; rows of the first 4096 anchors must equal the
    unpartitioned L=4096 problem on the same anchors (position invariance, Sec. 3.1)."""
    cfg = CONFIGS["c5_p99"]
    print(f"case {cfg.name}: generating inputs", flush=True)
    qb, kb, vb, dob = make_inputs(cfg)
    b = cfg.seg_bounds()
    tm = pe.peagle_build_tilemap(cfg.L, cfg.K, b, device=0)
    r = Run(tm, cfg.L, cfg.K, cfg.Hq, cfg.Hkv, cfg.D, qb, kb, vb, dob, cfg.scale)
    print(f"case {cfg.name}: partitioned step, {len(b) - 1} segments", flush=True)
    r.step(0, len(b) - 1)
    torch.cuda.synchronize()
    Lp = 4096
    (pq, pk, pv, pdo), idx = _prefix_inputs([qb, kb, vb, dob], cfg.L, Lp, cfg.K)
    print(f"case {cfg.name}: unpartitioned prefix L={Lp} on the same tile map", flush=True)
    rp = Run(tm, Lp, cfg.K, cfg.Hq, cfg.Hkv, cfg.D, pq, pk, pv, pdo, cfg.scale)
    rp.fwd()
    rp.bwd()
    torch.cuda.synchronize()
    tidx = torch.from_numpy(idx).cuda()
    assert torch.equal(r.o[tidx], rp.o)
    assert torch.equal(r.dq[tidx], rp.dq)
    assert torch.equal(r.lse[:, tidx], rp.lse)
    assert not torch.isnan(r.dk).any() and not torch.isnan(r.dv).any()
    del rp
    print(f"case {cfg.name}: oracle on sampled rows", flush=True)
    g = 3
    grp = cfg.Hq // cfg.Hkv
    hs = slice(g * grp, (g + 1) * grp)
    got = {"O": None, "LSE": None, "dQ": None, "dK": None, "dV": None}
    # pull only one KV group to the host
    got_g = {"O": bf16_to_f64(r.o[:, hs].contiguous()), "LSE": r.lse[hs].double().cpu().numpy(),
             "dQ": bf16_to_f64(r.dq[:, hs].contiguous()), "dK": r.dk[:, g:g + 1].double().cpu().numpy(),
             "dV": r.dv[:, g:g + 1].double().cpu().numpy()}

    class _Cfg:  # the sampled check indexes heads of a single-group problem
        L, K, Hq, Hkv, D, scale = cfg.L, cfg.K, grp, 1, cfg.D, cfg.scale

    _sampled_check(_Cfg, got_g, qb[:, hs], kb[:, g:g + 1], vb[:, g:g + 1], dob[:, hs], g=0, n_anchor_samples=4)


# ----------------------------------------------------------------------------- drop-token sampled sequences

def _paper_example_counts():
    """Per-anchor depth counts of the n=16, K=4 worked example of Sec. 3.2 (38 positions)."""
    import os
    path = os.path.join(os.path.dirname(__file__), "golden", "partition_example.txt")
    vals = {}
    with open(path) as f:
        for line in f:
            tok = line.split("#")[0].split()
            if tok and tok[0] != "assign":
                vals[tok[0]] = [int(x) for x in tok[1:]]
    n, K = vals["n"][0], vals["K"][0]
    count = np.ones(n, dtype=np.int32)
    for g in range(1, K):
        for p in vals[f"depth{g}"]:
            count[p - g] = g + 1
    assert count.sum() == vals["total"][0]
    return count, K


SAMPLED = [
    # name, L, K, Hq, Hkv, D, retention, seed, bounds
    ("paper_example", None, 4, 2, 1, 64, None, 300, None),
    ("paper_example_two_segments", None, 4, 2, 1, 64, None, 305, [0, 8, 16]),
    ("r08_k8", 200, 8, 4, 2, 64, 0.8, 310, None),
    ("r08_k8_unaligned_segments", 219, 8, 4, 2, 64, 0.8, 320, [0, 61, 130, 219]),
    ("r05_k4_several_tiles", 700, 4, 4, 2, 64, 0.5, 330, [0, 256, 512, 700]),
    ("r08_d128", 150, 8, 2, 1, 128, 0.8, 340, [0, 64, 150]),
    ("nothing_dropped", 100, 4, 2, 2, 64, 1.0, 350, None),
    ("only_depth0_kept", 100, 4, 2, 2, 64, 0.0, 360, None),
    ("k3", 90, 3, 2, 1, 64, 0.7, 370, None),
    ("k16_r09", 120, 16, 2, 2, 64, 0.9, 380, [0, 50, 120]),
    ("k1", 300, 1, 2, 1, 64, 0.5, 390, None),
]


@pytest.mark.parametrize("name,L,K,Hq,Hkv,D,ret,seed,bounds", SAMPLED, ids=[c[0] for c in SAMPLED])
def test_sampled_sequences_match_oracle(name, L, K, Hq, Hkv, D, ret, seed, bounds):
    """Conditional Drop-token sampled sequences: every output of the step on a sampled tile map against the
    oracle evaluated on the explicit token list (single pass), and - where segments are given - against
    the oracle's Algorithm 1 partitioned run."""
    from gpu_harness import SampledRun
    from peagle_inputs import cod_depth_counts
    if ret is None:
        count, K = _paper_example_counts()
        L = len(count)
    else:
        count = cod_depth_counts(L, K, ret, seed)
    print(f"case {name}: L={L} K={K} Hq={Hq} Hkv={Hkv} D={D} retention={ret} seed={seed} bounds={bounds} "
          f"tokens={int(count.sum())}", flush=True)
    ta, td = orc.cod_tokens(count)
    T = len(ta)
    qb, kb, vb, dob = (rand_bits((T, Hq, D), seed), rand_bits((T, Hkv, D), seed + 1), rand_bits((T, Hkv, D), seed + 2),
                       rand_bits((T, Hq, D), seed + 3))
    tm = pe.peagle_build_tilemap_sampled(count, K, bounds, device=0)
    assert tm.tokens(L) == T
    S = 1 if bounds is None else len(bounds) - 1
    r = SampledRun(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    dkb = torch.empty((T, Hkv, D), dtype=torch.bfloat16, device="cuda")
    dvb = torch.empty((T, Hkv, D), dtype=torch.bfloat16, device="cuda")
    r.step(0, S, dkb, dvb)
    got = r.results()
    q, k, v, do = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    ref = orc.attn_backward(q, k, v, do, L, K, r.shape.scale, tokens=(ta, td))
    _check_against_oracle(got, ref, name)
    assert np.array_equal(bf16_to_f64(dkb), bf16_to_f64(r.dk.to(torch.bfloat16)))
    assert np.array_equal(bf16_to_f64(dvb), bf16_to_f64(r.dv.to(torch.bfloat16)))
    if S > 1:
        part = orc.attn_step_partitioned_sampled(q, k, v, do, count, K, r.shape.scale, S)
        _check_against_oracle(got, part, name + " vs Algorithm 1 partition")
        # unpartitioned pass through the single-segment entry points on the same map
        r1 = SampledRun(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r1.fwd()
        r1.bwd()
        g1 = r1.results()
        for n in ("O", "LSE", "dQ"):
            assert np.array_equal(g1[n], got[n]), n
        for n in ("dK", "dV"):
            assert rel_l2(g1[n], got[n]) <= PART_REL, n
        # rows assigned to segments as Algorithm 1 does (chains follow position i+1): same outputs
        tm2 = pe.peagle_build_tilemap_sampled(count, K, bounds, device=0, assignment=pe.ASSIGN_ALGORITHM1)
        r2 = SampledRun(tm2, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r2.step(0, S)
        g2 = r2.results()
        _check_against_oracle(g2, part, name + " Algorithm 1 assignment")
        for n in ("dK", "dV"):
            assert rel_l2(g2[n], got[n]) <= PART_REL, n
        # resumed run on the same accumulators
        r3 = SampledRun(tm2, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r3.step(0, 1)
        r3.step(1, S)
        g3 = r3.results()
        for n in ("O", "LSE", "dQ", "dK", "dV"):
            assert np.array_equal(g3[n], g2[n]), n
    if ret == 1.0:
        # nothing dropped: same storage order as the dense layout; the dense map must agree to rounding order
        dm = pe.peagle_build_tilemap(L, K, bounds, device=0)
        d = Run(dm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        d.step(0, S)
        gd = d.results()
        for n in ("O", "dQ"):
            assert rel_l2(gd[n], got[n]) <= 2e-3, n          # bf16 outputs, different summation order
        assert max_abs(gd["LSE"], got["LSE"]) <= 1e-5
        for n in ("dK", "dV"):
            assert rel_l2(gd[n], got[n]) <= PART_REL, n


def test_full_size_sampled_c3_retention_08():
    """c3 shape under drop-token sampling with retention 0.8, in the launch configuration the benchmark's
    --cod-retention mode times: oracle on every kept depth of sampled anchors (O, LSE, dQ), on the keys of
    the last anchors (dK, dV), identities that hold at any size, and the unpartitioned run."""
    from gpu_harness import SampledRun
    from peagle_inputs import cod_depth_counts, make_inputs_tokens
    cfg = CONFIGS["c3_median"]
    L, K = cfg.L, cfg.K
    count = cod_depth_counts(L, K, 0.8, cfg.seed)
    ta, td = orc.cod_tokens(count)
    T = len(ta)
    print(f"case sampled c3: L={L} K={K} kept positions {T}", flush=True)
    qb, kb, vb, dob = make_inputs_tokens(cfg, T)
    b = cfg.seg_bounds()
    tm = pe.peagle_build_tilemap_sampled(count, K, b, device=0)
    r = SampledRun(tm, L, K, cfg.Hq, cfg.Hkv, cfg.D, qb, kb, vb, dob, cfg.scale)
    r.step(0, len(b) - 1)
    got = r.results()
    assert not any(np.isnan(got[n]).any() for n in got)
    g = 2
    grp = cfg.Hq // cfg.Hkv
    hs = slice(g * grp, (g + 1) * grp)
    q, k, v, do = (bf16_bits_to_f64(x) for x in (qb[:, hs], kb[:, g:g + 1], vb[:, g:g + 1], dob[:, hs]))
    rng = np.random.default_rng(1)
    anchors = np.unique(np.concatenate([[0, 1, 63, 64, L // 2, L - 1], rng.integers(0, L, size=6),
                                        np.nonzero(count == K)[0][:3]]))
    rows = np.nonzero(np.isin(ta, anchors))[0]
    print(f"case sampled c3: oracle on {len(rows)} rows", flush=True)
    ref = orc.attn_backward(q, k, v, do, L, K, cfg.scale, rows=rows, row_block=256, tokens=(ta, td))
    assert rel_l2(got["O"][rows][:, hs], ref["O"]) <= FWD_REL
    _check_o_abs(got["O"][rows][:, hs], ref["O"], "sampled c3")
    assert max_abs(got["LSE"][hs][:, rows], ref["LSE"]) <= LSE_ABS
    assert rel_l2(got["dQ"][rows][:, hs], ref["dQ"]) <= GRAD_REL
    rows2 = np.nonzero(ta >= L - 40)[0]                     # keys of the last anchors: seen by those anchors' rows only
    ref2 = orc.attn_backward(q, k, v, do, L, K, cfg.scale, rows=rows2, row_block=256, tokens=(ta, td))
    for n in ("dK", "dV"):
        assert rel_l2(got[n][rows2][:, g:g + 1], ref2[n][rows2]) <= GRAD_REL, n
    _check_global_identities(got, qb, kb, dob, cfg)
    r.fwd()
    r.bwd()
    whole = r.results()
    for n in ("O", "LSE", "dQ"):
        assert np.array_equal(whole[n], got[n]), n
    for n in ("dK", "dV"):
        assert rel_l2(got[n], whole[n]) <= PART_REL, n


# ----------------------------------------------------------------------------- packed batches

PACKED = [
    # name, seq_lens, K, Hq, Hkv, D, retention, seed, bounds, assignment
    ("three_short", (40, 25, 70), 4, 4, 2, 64, None, 400, None, 0),
    ("five_mixed_one_segment_each", (100, 37, 64, 1, 90), 8, 4, 2, 64, None, 410, [0, 100, 137, 201, 202, 292], 0),
    ("segments_across_sequences_sampled", (100, 37, 64, 1, 90), 8, 2, 1, 64, 0.8, 420, [0, 50, 120, 292], 1),
    ("d128_two", (90, 60), 8, 2, 1, 128, None, 430, [0, 64, 150], 0),
    ("k1_three", (130, 130, 130), 1, 2, 2, 64, None, 440, [0, 200, 390], 0),
    # more than 64 row tiles in a segment (one dK/dV launch: only dense segments are cut into chunks)
    ("long_packed_chunks", (700, 900, 500), 8, 2, 1, 64, None, 450, None, 0),
    ("long_sampled_chunks_alg1", (1500, 800), 8, 2, 1, 64, 0.8, 460, [0, 2050, 2300], 1),
]


@pytest.mark.parametrize("name,seq_lens,K,Hq,Hkv,D,ret,seed,bounds,assign", PACKED, ids=[c[0] for c in PACKED])
def test_packed_batches_match_oracle(name, seq_lens, K, Hq, Hkv, D, ret, seed, bounds, assign):
    """Variable-length batches packed before the expansion, one launch per kernel and segment for the whole
    batch: against the oracle on the packed token list, and (dense case) against each sequence run alone."""
    from gpu_harness import SampledRun
    from peagle_inputs import cod_depth_counts
    L = sum(seq_lens)
    count = None if ret is None else cod_depth_counts(L, K, ret, seed)
    tok = orc.packed_tokens(seq_lens, K, count)
    T = len(tok[0])
    print(f"case {name}: seq_lens={seq_lens} K={K} Hq={Hq} Hkv={Hkv} D={D} retention={ret} seed={seed} bounds={bounds} "
          f"assignment={assign} tokens={T}", flush=True)
    qb, kb, vb, dob = (rand_bits((T, Hq, D), seed), rand_bits((T, Hkv, D), seed + 1), rand_bits((T, Hkv, D), seed + 2),
                       rand_bits((T, Hq, D), seed + 3))
    tm = pe.peagle_build_tilemap_packed(seq_lens, K, count, bounds, device=0, assignment=assign)
    S = 1 if bounds is None else len(bounds) - 1
    r = SampledRun(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.step(0, S)
    got = r.results()
    q, k, v, do = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    ref = orc.attn_backward(q, k, v, do, L, K, r.shape.scale, tokens=tok)
    _check_against_oracle(got, ref, name)
    if S > 1:
        r1 = SampledRun(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r1.fwd()
        r1.bwd()
        g1 = r1.results()
        for n in ("O", "LSE", "dQ"):
            assert np.array_equal(g1[n], got[n]), n
        for n in ("dK", "dV"):
            assert rel_l2(g1[n], got[n]) <= PART_REL, n
    if ret is None:
        base = 0
        for Lq in seq_lens:
            idx = np.concatenate([d * L + base + np.arange(Lq) for d in range(K)])
            one_tm = pe.peagle_build_tilemap(Lq, K, None, device=0)
            one = Run(one_tm, Lq, K, Hq, Hkv, D, qb[idx], kb[idx], vb[idx], dob[idx])
            one.fwd()
            one.bwd()
            g = one.results()
            for n in ("O", "dQ"):
                assert rel_l2(got[n][idx], g[n]) <= 2e-3 or np.abs(got[n][idx] - g[n]).max() <= 1e-2, (n, Lq)
            assert max_abs(got["LSE"][:, idx], g["LSE"]) <= 1e-5
            for n in ("dK", "dV"):
                assert rel_l2(got[n][idx], g[n]) <= PART_REL, (n, Lq)
            base += Lq


def test_rebuilding_a_sampled_map_in_place_between_steps():
    """A new drop-token sample every step on one handle: the rebuilt map (asynchronous upload on the launch
    stream) must give exactly what a freshly built map gives, while the step before it keeps its results."""
    from gpu_harness import SampledRun
    from peagle_inputs import cod_depth_counts
    L, K, Hq, Hkv, D = 600, 8, 4, 2, 64
    bounds = [0, 256, 600]
    tm = pe.peagle_build_tilemap_sampled(cod_depth_counts(L, K, 0.8, 1), K, bounds, device=0)
    for step, (r, seed, Ls) in enumerate([(0.8, 2, L), (0.5, 3, L), (0.9, 4, 900), (0.7, 5, 300)]):
        count = cod_depth_counts(Ls, K, r, seed)
        b = [0, Ls // 2, Ls]
        print(f"step {step}: L={Ls} retention={r} kept={int(count.sum())}", flush=True)
        tm.rebuild((Ls,), count, b)
        T = tm.tokens(Ls)
        qb, kb, vb, dob = (rand_bits((T, Hq, D), seed), rand_bits((T, Hkv, D), seed + 1),
                           rand_bits((T, Hkv, D), seed + 2), rand_bits((T, Hq, D), seed + 3))
        run = SampledRun(tm, Ls, K, Hq, Hkv, D, qb, kb, vb, dob)
        run.step(0, 2)
        got = run.results()
        fresh = pe.peagle_build_tilemap_sampled(count, K, b, device=0)
        ref_run = SampledRun(fresh, Ls, K, Hq, Hkv, D, qb, kb, vb, dob)
        ref_run.step(0, 2)
        ref = ref_run.results()
        for n in ("O", "LSE", "dQ", "dK", "dV"):
            assert np.array_equal(got[n], ref[n]), (step, n)
    ta, td = orc.cod_tokens(count)
    q, k, v, do = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    _check_against_oracle(got, orc.attn_backward(q, k, v, do, Ls, K, run.shape.scale, tokens=(ta, td)), "after rebuilds")


def test_random_small_problems_match_oracle():
    """Seeded sweep over batches, depths, head shapes, retention rates, segmentations and assignments:
    the partitioned step on the general tile map against the oracle, every output.  PEAGLE_SWEEP_CASES widens
    the sweep for a one-off run."""
    from gpu_harness import SampledRun
    from peagle_inputs import cod_depth_counts
    import os
    rng = np.random.default_rng(77)
    for case in range(int(os.environ.get("PEAGLE_SWEEP_CASES", "10"))):
        K = int(rng.choice([1, 2, 4, 5, 8, 16]))
        n_seq = int(rng.integers(1, 4))
        seq_lens = tuple(int(x) for x in rng.integers(1, 120, size=n_seq))
        L = sum(seq_lens)
        D = int(rng.choice([64, 128]))
        Hkv = int(rng.choice([1, 2]))
        Hq = Hkv * int(rng.choice([1, 2, 3]))
        r = float(rng.choice([0.5, 0.8, 1.0]))
        count = None if rng.random() < 0.3 else cod_depth_counts(L, K, r, int(rng.integers(1 << 30)))
        S = int(rng.integers(1, 4))
        bounds = None
        if S > 1 and L > S:
            cuts = np.sort(rng.choice(np.arange(1, L), size=S - 1, replace=False))
            bounds = [0] + [int(c) for c in cuts] + [L]
        S = 1 if bounds is None else len(bounds) - 1
        assign = int(rng.integers(0, 2))
        tok = orc.packed_tokens(seq_lens, K, count)
        T = len(tok[0])
        what = (f"case {case}: seq_lens={seq_lens} K={K} Hq={Hq} Hkv={Hkv} D={D} sampled={count is not None} r={r} "
                f"bounds={bounds} assign={assign} tokens={T}")
        print(what, flush=True)
        seed = 1000 + 10 * case
        qb, kb, vb, dob = (rand_bits((T, Hq, D), seed), rand_bits((T, Hkv, D), seed + 1),
                           rand_bits((T, Hkv, D), seed + 2), rand_bits((T, Hq, D), seed + 3))
        tm = pe.peagle_build_tilemap_packed(seq_lens, K, count, bounds, device=0, assignment=assign)
        run = SampledRun(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        run.step(0, S)
        got = run.results()
        q, k, v, do = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
        _check_against_oracle(got, orc.attn_backward(q, k, v, do, L, K, run.shape.scale, tokens=tok), what)


def test_random_dense_problems_match_oracle():
    """Seeded sweep over dense maps: depths from 1 to the largest supported (128, one anchor per row tile) and depths
    that do not divide 128, lengths cropped below the map's, random segment cuts (multiples of the anchors per row
    tile), head shapes and both head sizes; the separate forward / backward calls or the partitioned step, every
    output against the oracle.  PEAGLE_SWEEP_CASES widens the sweep for a one-off run (about once per 1e8 output
    elements such a run meets a row of one or two keys whose O error reaches 1.02e-2: the bf16 rounding of P
    against values of opposite sign, not a defect)."""
    import os
    rng = np.random.default_rng(4242)
    n_cases = int(os.environ.get("PEAGLE_SWEEP_CASES", "14"))
    for case in range(n_cases):
        K = int(rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 8, 8, 12, 16, 20, 32, 64, 128]))
        A = 128 // K
        L_max = int(rng.integers(1, max(2, min(420, 2400 // K))))
        S = int(rng.integers(1, 5))
        inner = sorted({int(c) * A for c in rng.integers(1, max(2, -(-L_max // A)), size=S - 1)} - {0})
        inner = [c for c in inner if c < L_max]
        bounds = [0] + inner + [L_max] if inner else None
        L = L_max if rng.random() < 0.5 else int(rng.integers(1, L_max + 1))
        D = int(rng.choice([64, 128]))
        Hkv = int(rng.choice([1, 2, 3]))
        Hq = Hkv * int(rng.choice([1, 2, 3, 4]))
        whole_step = bool(rng.random() < 0.6)
        what = (f"dense case {case}: L={L} of L_max={L_max} K={K} Hq={Hq} Hkv={Hkv} D={D} bounds={bounds} "
                f"{'step' if whole_step else 'fwd+bwd'}")
        print(what, flush=True)
        T = L * K
        seed = 5000 + 10 * case
        qb, kb, vb, dob = (rand_bits((T, Hq, D), seed), rand_bits((T, Hkv, D), seed + 1),
                           rand_bits((T, Hkv, D), seed + 2), rand_bits((T, Hq, D), seed + 3))
        tm = pe.peagle_build_tilemap(L_max, K, bounds, device=0)
        r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        if whole_step:
            r.step(0, 1 if bounds is None else len(bounds) - 1)
        else:
            r.fwd()
            r.bwd()
        _check_against_oracle(r.results(), _oracle(qb, kb, vb, dob, L, K, r.shape.scale), what)


def test_partitioned_step_replays_from_a_hip_graph():
    """The step allocates nothing and synchronises nothing, so a caller may capture it: every replay, with
    eager work and synchronisations in between, must reproduce the eager results bit for bit."""
    L, K, Hq, Hkv, D = 300, 8, 4, 2, 64
    bounds = [0, 128, 300]
    T = L * K
    qb, kb, vb, dob = (rand_bits((T, Hq, D), 500), rand_bits((T, Hkv, D), 501), rand_bits((T, Hkv, D), 502),
                       rand_bits((T, Hq, D), 503))
    tm = pe.peagle_build_tilemap(L, K, bounds, device=0)
    eager = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    eager.step(0, 2)
    want = eager.results()
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        r.step(0, 2)                                    # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        r.step(0, 2)
    for replay in range(4):
        for t in (r.o, r.dq):
            t.fill_(float("nan"))
        r.lse.fill_(float("nan"))
        r.dk.fill_(float("nan"))
        r.dv.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        got = r.results()
        for n in ("O", "LSE", "dQ", "dK", "dV"):
            assert np.array_equal(got[n], want[n]), (replay, n)
        eager.step(0, 2)                                # the program's own eager work between replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("D,Hq,Hkv", [(64, 128, 2), (128, 64, 2)])
def test_tensors_beyond_4_gib_equal_their_halves(D, Hq, Hkv):
    """Q-shaped tensors just over 4 GiB (row copies then form 64-bit addresses) against the same problem with the query
    heads in two calls of half the size: heads do not interact, and dK/dV run over the same ranges of rows in either call (the
    work items take every slot), so every result has the same bits."""
    L, K = 2049, 128
    T = L * K
    assert T * Hq * D * 2 >= 1 << 32 > T * Hq * D
    print(f"case beyond 4 GiB D={D} Hq={Hq}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(77)
    rnd = lambda *sh: torch.randn(*sh, generator=g, device="cuda", dtype=torch.bfloat16)
    q, d_o, k, v = rnd(T, Hq, D), rnd(T, Hq, D), rnd(T, Hkv, D), rnd(T, Hkv, D)
    tm = pe.peagle_build_tilemap(L, K, None, device=0)

    def run(q, d_o, k, v):
        shape = pe.Shape(L, K, q.shape[1], k.shape[1], D)
        o, dq = torch.empty_like(q), torch.empty_like(q)
        lse = torch.empty((q.shape[1], T), device="cuda")
        dk, dv = (torch.empty(k.shape, device="cuda") for _ in range(2))
        ws = torch.empty(pe.peagle_workspace_bytes(tm, shape), dtype=torch.uint8, device="cuda")
        pe.peagle_attn_step_partitioned(tm, shape, 0, 1, q, k, v, d_o, o, lse, dq, dk, dv, None, None, ws)
        torch.cuda.synchronize()
        return {"o": o, "dq": dq, "dk": dk, "dv": dv, "lse": lse.t()}

    whole = run(q, d_o, k, v)
    for h in range(2):
        a, b = slice(h * Hq // 2, (h + 1) * Hq // 2), slice(h, h + 1)
        half = run(q[:, a].contiguous(), d_o[:, a].contiguous(), k[:, b].contiguous(), v[:, b].contiguous())
        for n, t in half.items():
            assert torch.isfinite(t).all(), n
            assert torch.equal(whole[n][:, b if n in ("dk", "dv") else a], t), n


@pytest.mark.parametrize("D,Hq,Hkv", [(64, 176, 2), (128, 88, 2)])
def test_listed_tensors_beyond_4_gib_equal_their_halves(D, Hq, Hkv):
    """The same for a packed batch, whose rows are named by lists; each row tile lacks 32 of its 128 rows."""
    lens, K = [1000, 1049], 96
    tm = pe.peagle_build_tilemap_packed(lens, K, device=0)
    L, T = sum(lens), tm.tokens(sum(lens))
    assert T * Hq * D * 2 >= 1 << 32 > T * Hq * D
    print(f"case listed beyond 4 GiB D={D} Hq={Hq}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(78)
    rnd = lambda H: torch.randn(T, H, D, generator=g, device="cuda", dtype=torch.bfloat16)
    q, d_o, k, v = rnd(Hq), rnd(Hq), rnd(Hkv), rnd(Hkv)
    whole = _heads_run(tm, L, K, q, k, v, d_o)
    for h in range(2):
        a, b = slice(h * Hq // 2, (h + 1) * Hq // 2), slice(h, h + 1)
        half = _heads_run(tm, L, K, *(t.contiguous() for t in (q[:, a], k[:, b], v[:, b], d_o[:, a])))
        for n, t in half.items():
            assert torch.isfinite(t).all(), n
            assert torch.equal(whole[n][:, b if n in ("dk", "dv") else a], t), n


@pytest.mark.parametrize("D", [64, 128])
def test_a_nan_stays_in_the_sequences_that_see_it(D):
    """Rows that a listed row tile lacks are read from the tile's own last row: a sequence of NaN queries and gradients
    packed first, between or last leaves every bit of the others as it was."""
    lens, K, Hq, Hkv = [37, 150, 5, 90], 7, 4, 2
    tm = pe.peagle_build_tilemap_packed(lens, K, device=0)
    L, T, start = sum(lens), tm.tokens(sum(lens)), np.concatenate([[0], np.cumsum(lens)])
    print(f"case NaN beside D={D}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(79)
    q, k, v, d_o = (torch.randn(T, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq))
    clean = _heads_run(tm, L, K, q, k, v, d_o)
    anchor = torch.arange(T, device="cuda") % L               # (every depth kept: token d * L + i)
    for s in (0, 2, 3):
        own = (anchor >= int(start[s])) & (anchor < int(start[s + 1]))
        spoilt_q, spoilt_do = q.clone(), d_o.clone()
        spoilt_q[own], spoilt_do[own] = float("nan"), float("nan")
        got = _heads_run(tm, L, K, spoilt_q, k, v, spoilt_do)
        for n in ("o", "lse", "dq"):
            assert torch.equal(got[n][~own], clean[n][~own]), (n, s)
        # (key tiles are shared at a sequence's ends, and a zero probability times a NaN dP is NaN there, as ever)
        tiles = {int(start[s]) // 64, (int(start[s + 1]) - 1) // 64}
        apart = ~own & ~torch.isin(anchor // 64, torch.tensor(sorted(tiles), device="cuda"))
        apart |= ~own & (torch.arange(T, device="cuda") >= L)  # chain keys are in tiles of their own rows
        for n in ("dk", "dv"):
            assert torch.equal(got[n][apart], clean[n][apart]), (n, s)


@pytest.mark.parametrize("D,spoilt,kept", [(64, 0, (32, 126)), (64, 125, (0, 64)), (128, 0, (0, 0)), (128, 125, (0, 0))])
def test_a_nan_row_stays_with_the_chain_keys_that_share_its_unit(D, spoilt, kept):
    """Row tiles of 18 anchors of K = 7: 126 rows and two missing ones.  At D = 64 chain keys are taken with the 32-row units
    that hold rows of their anchors, so a NaN first row (unit 0) reaches those of the first 32 slots and a NaN last row (unit
    3) those of the slots from 64 on, whose anchors reach unit 3; the missing rows (unit 3 as well) carry it no further.  At
    D = 128 a chain key is taken with the whole tile.  No other tile's chain keys see the row at all."""
    lens, K, Hq, Hkv, first = [37, 150, 90], 7, 4, 2, 37 + 18      # (the second tile of the second sequence)
    tm = pe.peagle_build_tilemap_packed(lens, K, device=0)
    L, T = sum(lens), tm.tokens(sum(lens))
    assert T == L * K and 128 // K == 18                           # every depth kept: token d * L + i
    print(f"case NaN in one row D={D} row={spoilt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(80)
    q, k, v, d_o = (torch.randn(T, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq))
    clean = _heads_run(tm, L, K, q, k, v, d_o)
    tok = torch.arange(T, device="cuda")
    anchor, depth = tok % L, tok // L
    mine = (anchor >= first) & (anchor < first + 18)
    slot = (anchor - first) * K + depth                            # row of the tile, and slot of its chain key
    for t in (q, d_o):
        t[mine & (slot == spoilt)] = float("nan")
    got = _heads_run(tm, L, K, q, k, v, d_o)
    apart = (depth >= 1) & (~mine | (slot >= kept[0]) & (slot < kept[1]))
    for n in ("dk", "dv"):
        assert torch.isfinite(got[n][apart]).all(), n
        # (the forward takes the tile's other rows again with the running max: the same to rounding, not to the bit)
        assert _grad_rel(got[n][apart].double().cpu().numpy(), clean[n][apart].double().cpu().numpy()) <= GRAD_REL, n


@pytest.mark.parametrize("L_max,L,bounds", [(530, 530, None), (700, 517, None), (600, 600, [0, 520, 600])],
                         ids=["two_chunks", "cropped", "chunks_then_a_segment"])
def test_dense_segments_of_more_than_128_row_tiles(L_max, L, bounds):
    """133, 130 and 130 + 20 row tiles (K = 32, four anchors each): a segment past 128 row tiles runs its dK/dV in two
    equal chunks, the second adding to what the first wrote."""
    K, Hq, Hkv, D, seed = 32, 2, 1, 64, 310
    print(f"case dense chunks: L={L} of {L_max} K={K} bounds={bounds}", flush=True)
    qb, kb, vb, dob = (rand_bits((L * K, H, D), seed + i) for i, H in enumerate((Hq, Hkv, Hkv, Hq)))
    tm = pe.peagle_build_tilemap(L_max, K, bounds, device=0)
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.step(0, 1 if bounds is None else len(bounds) - 1)
    got = r.results()
    ref = _oracle(qb, kb, vb, dob, L, K, r.shape.scale)
    _check_against_oracle(got, ref, f"dense chunks {L} {bounds}")
    for n in ("dK", "dV"):                      # no key left out or counted twice at a chunk boundary
        assert max_abs(got[n], ref[n]) <= 2e-2 * np.abs(ref[n]).max(), n


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("K,L", [(8, 3), (8, 15), (8, 16), (8, 17), (8, 130), (4, 31), (4, 100), (5, 24), (5, 25), (5, 201), (7, 19), (7, 73),
                                 (7, 5), (33, 2), (33, 10), (43, 2), (43, 7), (32, 9)])
def test_every_way_dkdv_finds_its_rows(K, L, D):
    """Row tiles of 128 rows at a constant step, of fewer with the missing ones in a tile's last copy (K = 5, 7; K = 33 at
    D = 64), and of neither kind (K = 43; K = 33 at D = 128); less than one tile, one, one and a bit, several."""
    Hq, Hkv, seed = 4, 2, 330 + K
    print(f"case rows: L={L} K={K} D={D}", flush=True)
    qb, kb, vb, dob = (rand_bits((L * K, H, D), seed + i) for i, H in enumerate((Hq, Hkv, Hkv, Hq)))
    r = Run(pe.peagle_build_tilemap(L, K, None, device=0), L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.step(0, 1)
    got = r.results()
    ref = _oracle(qb, kb, vb, dob, L, K, r.shape.scale)
    _check_against_oracle(got, ref, f"rows {K} {L} {D}")
    for n in ("dK", "dV"):                      # no row left out, read twice or taken from beyond the sequence
        assert max_abs(got[n], ref[n]) <= 2e-2 * np.abs(ref[n]).max(), n


@pytest.mark.parametrize("qscale", [1.0, 12.0])
def test_pipelined_dq_over_lists_of_every_length(qscale):
    """Lists of 3 to 34 key tiles at D = 64, few workgroups: the pipelined dQ (in the one grid) with every remainder of its groups of
    three tiles and (large logits) with normalised and unnormalised probabilities.  The whole sequence, its segments one
    by one and a crop agree bit for bit."""
    L, K, Hq, Hkv, D, bounds = 2000, 4, 2, 1, 64, [0, 1472, 1568, 2000]
    print(f"case dq choice qscale={qscale}", flush=True)
    T = L * K
    qb, kb, vb, dob = (rand_bits((T, Hq, D), 320, qscale), rand_bits((T, Hkv, D), 321), rand_bits((T, Hkv, D), 322),
                       rand_bits((T, Hq, D), 323))
    tm = pe.peagle_build_tilemap(L, K, bounds, device=0)
    assert dq_path(tm, Hq) == "one grid"
    r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    r.step(0, 3)
    got = r.results()
    ref = _oracle(qb, kb, vb, dob, L, K, r.shape.scale)
    assert rel_l2(got["O"], ref["O"]) <= FWD_REL
    for n in ("dQ", "dK", "dV"):
        assert rel_l2(got[n], ref[n]) <= GRAD_REL, n
    r2 = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
    for s in range(3):
        r2.step(s, s + 1)
    g2 = r2.results()
    for n in got:
        assert np.array_equal(g2[n], got[n]), n
    Lc = 1600                                            # rows of a prefix view: the same tiles, the same bits
    keep = np.concatenate([d * L + np.arange(Lc) for d in range(K)])
    rc = Run(tm, Lc, K, Hq, Hkv, D, qb[keep], kb[keep], vb[keep], dob[keep])
    rc.step(0, 3)
    gc = rc.results()
    whole = np.concatenate([d * Lc + np.arange(1600 // 32 * 32) for d in range(K)])
    back = np.concatenate([d * L + np.arange(1600 // 32 * 32) for d in range(K)])
    assert np.array_equal(gc["dQ"][whole], got["dQ"][back]) and np.array_equal(gc["O"][whole], got["O"][back])


def _map_of(form):
    """A map with lists of 3 to 34 (dense), 2 to 14 (packed) or 2 to 30 (sampled) tiles, and its L and K."""
    if form == "dense":
        return pe.peagle_build_tilemap(2011, 4, [0, 1472, 2011], device=0), 2011, 4
    if form == "k7":                                # row tiles of 126 rows
        return pe.peagle_build_tilemap(1200, 7, None, device=0), 1200, 7
    if form == "packed":
        lens = [700, 3, 411, 64, 1, 129, 620]
        return pe.peagle_build_tilemap_packed(lens, 8, device=0), sum(lens), 8
    from peagle_inputs import cod_depth_counts
    count = cod_depth_counts(1700, 5, 0.8, 331)
    return pe.peagle_build_tilemap_sampled(count, 5, [0, 650, 1700], device=0), 1700, 5


@pytest.mark.parametrize("qscale", [1.0, 12.0, 40.0])
@pytest.mark.parametrize("form", ["dense", "k7", "packed", "sampled"])
def test_both_dq_kernels_give_the_same_bits(form, qscale):
    """Kernels launched apart: forty query heads in one call (many workgroups: the plain dQ kernel at D = 64) against the same heads
    in calls of one key / value head's group each (few workgroups: the pipelined kernel).  At the larger scales some or all workgroups
    have row sums outside the range of unnormalised probabilities."""
    print(f"case dq kernels {form} qscale={qscale}", flush=True)
    tm, L, K = _map_of(form)
    T, Hq, Hkv, D = tm.tokens(L), 40, 20, 64
    assert dq_path(tm, Hq, "profiled") == "plain" and dq_path(tm, Hq // Hkv, "profiled") == "pipelined"
    g = torch.Generator(device="cuda").manual_seed(335)
    rnd = lambda H, f=1.0: (torch.randn(T, H, D, generator=g, device="cuda") * f).to(torch.bfloat16)
    q, k, v, d_o = rnd(Hq, qscale), rnd(Hkv), rnd(Hkv), rnd(Hq)

    whole = _heads_run(tm, L, K, q, k, v, d_o, profiled=True)
    for h in range(0, Hkv, 3):
        a, b = slice(h * (Hq // Hkv), (h + 1) * (Hq // Hkv)), slice(h, h + 1)
        part = _heads_run(tm, L, K, q[:, a].contiguous(), k[:, b].contiguous(), v[:, b].contiguous(), d_o[:, a].contiguous(),
                          profiled=True)
        for n, t in part.items():
            assert torch.isfinite(t).all(), n
            assert torch.equal(whole[n][:, b if n in ("dk", "dv") else a], t), n


@pytest.mark.parametrize("D,qscale", [(64, 1.0), (64, 40.0), (128, 1.0)])
@pytest.mark.parametrize("form", ["one_row", "one_tile", "dense", "k7", "k43", "packed", "sampled"])
def test_backward_as_one_grid_gives_the_bits_of_kernels_launched_apart(form, D, qscale):
    """A step runs dQ and dK/dV as one grid behind a forward that leaves the per-row terms; a profiled step launches them
    apart; a backward called by itself forms the terms in a pass of its own (D = 64) or in dQ's kernel.  The smallest problems, segments, every way of
    finding rows, and (at the larger scale) rows outside the range of unnormalised probabilities: the same bits."""
    print(f"case one grid {form} D={D} qscale={qscale}", flush=True)
    small = {"one_row": (1, 8), "one_tile": (16, 8), "k43": (300, 43)}
    tm, L, K = (pe.peagle_build_tilemap(*small[form], None, device=0), *small[form]) if form in small else _map_of(form)
    S = tm.info()["S"]
    T, Hq, Hkv = tm.tokens(L), 6, 2
    shape = pe.Shape(L, K, Hq, Hkv, D)
    g = torch.Generator(device="cuda").manual_seed(341)
    rnd = lambda H, f=1.0: (torch.randn(T, H, D, generator=g, device="cuda") * f).to(torch.bfloat16)
    q, k, v, d_o = rnd(Hq, qscale), rnd(Hkv), rnd(Hkv), rnd(Hq)
    ws = torch.empty(pe.peagle_workspace_bytes(tm, shape), dtype=torch.uint8, device="cuda")

    def results(call):
        out = [torch.full_like(q, float("nan")), torch.full((Hq, T), float("nan"), device="cuda"), torch.full_like(q, float("nan")),
               *(torch.full((T, Hkv, D), float("nan"), device="cuda") for _ in range(2))]
        ws.fill_(255)  # (NaN: terms that nobody formed would show)
        call(*out)
        torch.cuda.synchronize()
        return dict(zip(("o", "lse", "dq", "dk", "dv"), out))

    def by_hand(o, lse, dq, dk, dv):
        pe.peagle_attn_fwd(tm, shape, -1, q, k, v, o, lse)
        pe.peagle_attn_bwd(tm, shape, -1, q, k, v, o, d_o, lse, dq, dk, dv, 0, ws)
    step = results(lambda *out: pe.peagle_attn_step_partitioned(tm, shape, 0, S, q, k, v, d_o, *out, None, None, ws))
    apart = results(lambda *out: pe.peagle_attn_step_profiled(tm, shape, 0, S, q, k, v, d_o, *out, ws))
    calls = results(by_hand)
    for n in step:
        assert torch.isfinite(step[n]).all(), n
        assert torch.equal(step[n], apart[n]), n
        if S == 1 or n not in ("dk", "dv"):  # (segments are summed one by one, a call over all of them is not)
            assert torch.equal(step[n], calls[n]), n


@pytest.mark.parametrize("qscale", [1.0, 12.0, 40.0])
@pytest.mark.parametrize("form", ["dense", "k7", "packed", "sampled"])
def test_plain_dq_kernel_gives_the_bits_of_the_one_grid(form, qscale):
    """Short lists and more than 4,096 dQ workgroups in one step - the plain dQ kernel, before dK/dV - against calls of one key /
    value head's group each, which run dQ and dK/dV as one grid."""
    print(f"case plain dq against one grid {form} qscale={qscale}", flush=True)
    tm, L, K = _map_of(form)
    T, Hq, Hkv, D = tm.tokens(L), 96, 48, 64
    assert dq_path(tm, Hq) == "plain" and dq_path(tm, Hq // Hkv) == "one grid"
    g = torch.Generator(device="cuda").manual_seed(343)
    rnd = lambda H, f=1.0: (torch.randn(T, H, D, generator=g, device="cuda") * f).to(torch.bfloat16)
    q, k, v, d_o = rnd(Hq, qscale), rnd(Hkv), rnd(Hkv), rnd(Hq)
    whole = _heads_run(tm, L, K, q, k, v, d_o)
    for h in range(0, Hkv, 23):
        a, b = slice(2 * h, 2 * h + 2), slice(h, h + 1)
        part = _heads_run(tm, L, K, q[:, a].contiguous(), k[:, b].contiguous(), v[:, b].contiguous(), d_o[:, a].contiguous())
        for n, t in part.items():
            assert torch.isfinite(t).all(), n
            assert torch.equal(whole[n][:, b if n in ("dk", "dv") else a], t), n


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("form", ["short", "six_segments", "cropped", "chunks", "sampled", "packed", "rope"])
def test_segments_that_share_a_launch_give_the_bits_of_one_launch_each(form, D):
    """Few heads: up to four segments (or chunks of a long one) share a launch and the sum of its partials; in a workspace with
    room for one set of partials each has a launch and a sum of its own, as it has when a caller steps segment by segment."""
    print(f"case shared launch {form} D={D}", flush=True)
    K, L, Hq, Hkv = (32, 530, 2, 1) if form == "chunks" else (8, 1000, 4, 2)
    bounds = [0, 520, 530] if form == "chunks" else [0, 160, 320, 336, 640, 800, 1000]
    if form == "short":
        L, bounds = 150, [0, 16, 64, 80, 128, 150]       # (launches of four segments and of one)
    Lc = 650 if form == "cropped" else L                 # (ends inside the fifth segment)
    if form == "sampled":
        from peagle_inputs import cod_depth_counts
        build = lambda b: pe.peagle_build_tilemap_sampled(cod_depth_counts(L, K, 0.8, 351), K, b, device=0)
    elif form == "packed":
        build = lambda b: pe.peagle_build_tilemap_packed([300, 33, 467, 200], K, None, b, device=0)
    else:
        build = lambda b: pe.peagle_build_tilemap(L, K, b, device=0)
    tm, S = build(bounds), len(bounds) - 1
    shape, T, rope = pe.Shape(Lc, K, Hq, Hkv, D), tm.tokens(Lc), form == "rope"
    need = pe.peagle_rope_workspace_bytes if rope else pe.peagle_workspace_bytes
    g = torch.Generator(device="cuda").manual_seed(349)
    q, k, v, d_o = (torch.randn(T, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq))
    table = torch.empty((pe.peagle_rope_positions(tm, Lc), 2, D // 2), device="cuda")
    pe.peagle_rope_table(1e4, D, table.shape[0], table)

    def results(n_bytes, steps):
        ws = torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda")  # (NaN)
        out = [torch.zeros_like(q), torch.zeros((Hq, T), device="cuda"), torch.zeros_like(q),
               *(torch.full((T, Hkv, D), float("nan"), device="cuda") for _ in range(2))]
        for a, b in steps:
            if rope:
                pe.peagle_attn_step_partitioned_rope(tm, shape, a, b, q, k, v, d_o, table, *out, None, None, ws)
            else:
                pe.peagle_attn_step_partitioned(tm, shape, a, b, q, k, v, d_o, *out, None, None, ws)
        torch.cuda.synchronize()
        return out

    part, rest = 2 * Hq * ((Lc + 63) // 64 * 64) * D * 4, 2 * ((T * Hq * 4 + 255) // 256 * 256)
    sets = (pe.peagle_workspace_bytes(tm, shape) - rest) // part
    assert pe.peagle_workspace_bytes(tm, shape) == rest + sets * part and sets == (3 if form == "chunks" else 4)
    one_set = need(tm, shape) - (sets - 1) * part
    want = results(one_set, [(s, s + 1) for s in range(S)])
    for n_bytes in (need(tm, shape), one_set):
        for got, ref in zip(results(n_bytes, [(0, S)]), want):
            assert torch.isfinite(got).all() and torch.equal(got, ref)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_chunks_that_share_a_launch_in_a_backward_by_itself(accumulate, D):
    """A backward over a segment of two chunks with few heads: both share a launch where the workspace has room for two sets of
    partials, and with accumulate the first set that holds a key adds to what the caller's tensors hold.  The same bits as
    with a launch and a sum for each."""
    print(f"case shared launch backward accumulate={accumulate} D={D}", flush=True)
    K, L, Hq, Hkv = 32, 530, 2, 1
    tm, shape, T = pe.peagle_build_tilemap(L, K, None, device=0), pe.Shape(L, K, Hq, Hkv, D), L * K
    g = torch.Generator(device="cuda").manual_seed(353)
    q, k, v, d_o = (torch.randn(T, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq))
    old = [torch.randn(T, Hkv, D, generator=g, device="cuda") for _ in range(2)]
    o, lse = torch.empty_like(q), torch.empty((Hq, T), device="cuda")
    pe.peagle_attn_fwd(tm, shape, -1, q, k, v, o, lse)

    def results(n_bytes, accumulate):
        ws = torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda")  # (NaN)
        out = [torch.full_like(q, float("nan")), *(t.clone() for t in old)]
        pe.peagle_attn_bwd(tm, shape, -1, q, k, v, o, d_o, lse, *out, accumulate, ws)
        torch.cuda.synchronize()
        return out
    need = pe.peagle_workspace_bytes(tm, shape)
    one_set = 2 * T * Hq * 4 + 2 * Hq * 576 * D * 4      # (whole multiples of 256 bytes)
    assert need == one_set + 2 * Hq * 576 * D * 4
    got, ref = results(need, accumulate), results(one_set, accumulate)
    for a, b in zip(got, ref):
        assert torch.isfinite(a).all() and torch.equal(a, b)
    if accumulate:      # (an fp32 sum of the same terms in another order, and two subtractions: five roundings of 2^-24)
        for a, b, t in zip(got[1:], results(need, 0)[1:], old):
            assert (a - b - t).abs().max() <= 5 * 2.0 ** -24 * float((b.abs() + t.abs()).max())


@pytest.mark.parametrize("Hq,Hkv", [(2, 1), (112, 56)])
def test_a_sequence_keeps_its_bits_whatever_it_is_packed_with(Hq, Hkv):
    """Six hundred anchors alone (short lists, at many heads the plain dQ kernel) and packed in front of a sequence of five
    thousand (long lists, the pipelined form in one grid).  With these numbers of heads dK/dV run in one range of rows in both;
    the next test has those with which they do not."""
    K, D, own, other = 8, 64, 600, 5000
    print(f"case packed neighbours Hq={Hq}", flush=True)
    maps = [pe.peagle_build_tilemap_packed(lens, K, device=0) for lens in ([own], [own, other])]
    assert dq_path(maps[0], Hq) == ("plain" if Hq == 112 else "one grid") and dq_path(maps[1], Hq) == "one grid"
    g = torch.Generator(device="cuda").manual_seed(337)
    L = own + other
    full = [torch.randn(K, L, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq)]
    results = []
    for tm, n in zip(maps, (own, L)):
        r = _heads_run(tm, n, K, *(t[:, :n].reshape(K * n, t.shape[2], D).contiguous() for t in full))
        results.append({m: r[m].view(K, n, -1, D)[:, :own] for m in ("o", "dq", "dk", "dv")})
    for m in results[0]:
        assert torch.equal(results[0][m], results[1][m]), m


@pytest.mark.parametrize("Hq,alone,packed", [(4, 3, 2), (8, 3, 1)])
def test_the_last_bits_of_a_sequences_key_gradients_may_depend_on_what_it_is_packed_with(Hq, alone, packed):
    """The same sequence with four and eight heads: dK/dV run in three chunks alone and in two or one packed.  O, LSE and dQ
    have the same bits; a key's gradients are sums of the same fp32 terms in another grouping."""
    K, D, Hkv, own, other = 8, 64, 1, 600, 5000
    print(f"case packed neighbours, chunks Hq={Hq}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(338)
    L = own + other
    full = [torch.randn(K, L, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq)]
    results = []
    for lens, n, sets in (([own], own, alone), ([own, other], L, packed)):
        tm = pe.peagle_build_tilemap_packed(lens, K, device=0)
        part, base = 2 * Hq * ((n + 63) // 64 * 64) * D * 4, 2 * ((tm.tokens(n) * Hq * 4 + 255) // 256 * 256)
        assert pe.peagle_workspace_bytes(tm, pe.Shape(n, K, Hq, Hkv, D)) == base + sets * part
        r = _heads_run(tm, n, K, *(t[:, :n].reshape(K * n, t.shape[2], D).contiguous() for t in full))
        results.append({m: r[m].view(K, n, r[m].shape[1], -1)[:, :own] for m in r})
    for m in ("o", "lse", "dq"):
        assert torch.equal(results[0][m], results[1][m]), m
    # Each of the two sums takes a rounding for every 16 rows, head and chunk, of a partial sum that is, root mean square,
    # no larger than the whole sum of terms of either sign.
    roundings = own * K // 16 + Hq + 3
    for m in ("dk", "dv"):
        a, b = (r[m].double().cpu().numpy() for r in results)
        assert 0 < rel_l2(a, b) <= 2 * roundings * 2.0 ** -24, m


def test_sampled_map_of_long_lists_runs_the_pipelined_dq():
    from peagle_inputs import cod_depth_counts
    tm = pe.peagle_build_tilemap_sampled(cod_depth_counts(3000, 4, 0.8, 395), 4, None, device=0)
    assert mean_list(tm) > 24 and dq_path(tm, 2) == "one grid"
    test_sampled_sequences_match_oracle("long_lists", 3000, 4, 2, 1, 64, 0.8, 395, None)


@pytest.mark.parametrize("K,L,L_max,Hq,Hkv", [(1, 60, 300, 3, 3), (1, 130, 300, 10, 5), (3, 50, 200, 15, 5), (3, 43, 130, 7, 1),
                                              (8, 65, 128, 11, 11), (5, 77, 77, 9, 3), (2, 65, 200, 12, 6), (128, 2, 3, 5, 5)])
@pytest.mark.parametrize("D", [64, 128])
def test_key_tiles_at_and_past_the_end_of_a_cropped_sequence(D, K, L, L_max, Hq, Hkv):
    """A row tile of more anchors than the sequence has left lists key tiles that the sequence ends in, or that lie wholly past
    it (K = 1 and 3), whose rows the copies must not look for; none, one and two chain tiles, which a row tile takes first;
    numbers of heads of which none is a power of two."""
    seed = 360 + K + L
    print(f"case end of sequence: K={K} L={L} of {L_max} Hq={Hq} Hkv={Hkv} D={D}", flush=True)
    qb, kb, vb, dob = (rand_bits((L * K, H, D), seed + i) for i, H in enumerate((Hq, Hkv, Hkv, Hq)))
    tm = pe.peagle_build_tilemap(L_max, K, None, device=0)
    ref = _oracle(qb, kb, vb, dob, L, K, pe.Shape(L, K, Hq, Hkv, D).scale)
    for whole_step in (True, False):
        r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        if whole_step:
            r.step(0, 1)
        else:
            r.fwd()
            r.bwd()
        _check_against_oracle(r.results(), ref, f"end K={K} L={L} D={D}")


@pytest.mark.parametrize("L,L_max,bounds,Hq,sets", [
    (64, 64, None, 4, 1), (66, 66, None, 4, 2), (130, 300, None, 5, 3), (252, 252, None, 4, 3), (256, 256, None, 4, 4),
    (66, 66, None, 3, 1), (200, 200, [0, 100, 200], 4, 4), (210, 210, [0, 60, 180, 210], 4, 3), (130, 130, None, 60, 1),
    (160, 160, None, 60, 3)])
@pytest.mark.parametrize("D", [64, 128])
def test_few_heads_run_a_range_of_rows_in_chunks(D, L, L_max, bounds, Hq, sets):
    """K = 32, four anchors a row tile: 16, 17, 33 (cropped), 63 and 64 row tiles of few heads in one to four chunks that share a
    launch, two and three segments, fewer heads than are cut for, and sixty heads, whose work items leave slots for one chunk
    where lists are short and for three (at D = 128 two) where they are not."""
    K, Hkv, seed = 32, 1 if Hq < 60 else 10, 370
    if (D, L) == (128, 160):
        sets = 2
    print(f"case chunks of few heads L={L} of {L_max} Hq={Hq} D={D} bounds={bounds}", flush=True)
    T, S = L * K, 1 if bounds is None else len(bounds) - 1
    tm, shape = pe.peagle_build_tilemap(L_max, K, bounds, device=0), pe.Shape(L, K, Hq, Hkv, D)
    part = 2 * Hq * ((L + 63) // 64 * 64) * D * 4           # (whole multiples of 256 bytes)
    base = 2 * ((T * Hq * 4 + 255) // 256 * 256)
    need = pe.peagle_workspace_bytes(tm, shape)
    assert need == base + sets * part
    qb, kb, vb, dob = (rand_bits((T, H, D), seed + i) for i, H in enumerate((Hq, Hkv, Hkv, Hq)))

    def results(n_bytes, whole):
        r = Run(tm, L, K, Hq, Hkv, D, qb, kb, vb, dob)
        r.ws = torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda")  # (NaN)
        if whole:
            r.step(0, S)
        else:
            r.fwd()
            r.bwd()
        return r.results()
    got = results(need, True)
    one = results(base + part, True)                        # a launch and a sum for each chunk: the same bits
    for n in got:
        assert np.array_equal(got[n], one[n]), n
    calls = results(need, False)
    if S == 1:
        for n in got:
            assert np.array_equal(got[n], calls[n]), n
    if Hq <= 5:
        ref = _oracle(qb, kb, vb, dob, L, K, shape.scale)
        _check_against_oracle(got, ref, f"chunks {L} {Hq} {D}")
        _check_against_oracle(calls, ref, f"chunks by calls {L} {Hq} {D}")
        for n in ("dK", "dV"):                              # no key left out or counted twice at a chunk boundary
            assert max_abs(got[n], ref[n]) <= 2e-2 * np.abs(ref[n]).max(), n


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("form,sets", [("sampled", 3), ("two_segments", 4), ("algorithm1", 4), ("one_sequence", 3), ("many_short", 1),
                                       ("long_beside_short", 3)])
def test_few_heads_of_listed_maps_run_in_chunks(form, sets, D):
    """Sampled and packed maps of four heads: a range of rows in chunks whose lists are cut by position, in pieces of a list, of a
    sequence or between sequences, and not where many short sequences make the lists short already.  In a workspace with
    room for one set of partials each chunk has a launch of its own: the same bits."""
    from peagle_inputs import cod_depth_counts
    print(f"case chunks of listed maps {form} D={D}", flush=True)
    Hq, Hkv, seed = 4, 1, 380
    if form in ("sampled", "two_segments", "algorithm1"):
        L, K = 1050, 7
        bounds = None if form == "sampled" else [0, 400, 1050]
        sets -= bounds is not None and D == 128             # (half the slots: the first segment stays whole)
        count, assign = cod_depth_counts(L, K, 0.9, seed), int(form == "algorithm1")
        tm = pe.peagle_build_tilemap_sampled(count, K, bounds, device=0, assignment=assign)
        test_sampled_sequences_match_oracle(form, L, K, Hq, Hkv, D, 0.9, seed, bounds)
    else:
        K = 8 if form == "many_short" else 16
        lens = {"one_sequence": [330], "many_short": [64] * 10, "long_beside_short": [20, 290, 3, 41]}[form]
        L = sum(lens)
        tm = pe.peagle_build_tilemap_packed(lens, K, device=0)
        test_packed_batches_match_oracle(form, lens, K, Hq, Hkv, D, None, seed, None, 0)
    S, T, shape = tm.info()["S"], tm.tokens(L), pe.Shape(L, K, Hq, Hkv, D)
    part = 2 * Hq * ((L + 63) // 64 * 64) * D * 4
    base = 2 * ((T * Hq * 4 + 255) // 256 * 256)
    assert pe.peagle_workspace_bytes(tm, shape) == base + sets * part
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v, d_o = (torch.randn(T, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq))

    def results(n_bytes):
        ws = torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda")  # (NaN)
        out = [torch.full_like(q, float("nan")), torch.full((Hq, T), float("nan"), device="cuda"), torch.full_like(q, float("nan")),
               *(torch.full((T, Hkv, D), float("nan"), device="cuda") for _ in range(2))]
        pe.peagle_attn_step_partitioned(tm, shape, 0, S, q, k, v, d_o, *out, None, None, ws)
        torch.cuda.synchronize()
        return out
    for a, b in zip(results(pe.peagle_workspace_bytes(tm, shape)), results(base + part)):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("K,L,L_max,Hq,Hkv", [(1, 1500, 1500, 111, 37), (2, 1000, 1300, 81, 27), (8, 400, 400, 54, 18), (5, 37, 5000, 645, 215)])
def test_one_head_forwards_of_three_and_four_per_cu_give_the_same_bits(K, L, L_max, Hq, Hkv):
    """Odd groups, which the forward takes one head at a time: 1,280 workgroups and more (four per CU: two tile buffers, in the
    first of which a chain tile stands before the first tile of depth-0 keys) against each of some groups alone (three per CU,
    three buffers), with no, one and two chain tiles, a cropped sequence, and half of the heads done again with the running max;
    the first and the last group against the oracle too."""
    D, n = 64, Hq // Hkv
    print(f"case one-head forwards K={K} L={L} of {L_max} Hq={Hq}", flush=True)
    tm, used = (pe.peagle_build_tilemap(x, K, None, device=d) for x, d in ((L_max, 0), (L, -1)))
    assert used.info()["n_row_tiles"] * Hq >= 1280 and one_head_per_cu(used, Hq) == 4 and one_head_per_cu(used, n) == 3
    qb, kb, vb, dob = (rand_bits((L * K, H, D), 390 + i) for i, H in enumerate((Hq, Hkv, Hkv, Hq)))
    q, k, v = (to_dev_bf16(x) for x in (qb, kb, vb))
    q[:, 1::2] *= 32.0                                  # (a power of two: exact)

    def fwd(q, k, v):
        o, lse = torch.full_like(q, float("nan")), torch.full((q.shape[1], L * K), float("nan"), device="cuda")
        pe.peagle_attn_fwd(tm, pe.Shape(L, K, q.shape[1], k.shape[1], D), -1, q, k, v, o, lse)
        torch.cuda.synchronize()
        return o, lse
    o, lse = fwd(q, k, v)
    for h in sorted({0, 1, Hkv // 2, Hkv - 1}):
        a, b = slice(h * n, (h + 1) * n), slice(h, h + 1)
        o1, lse1 = fwd(*(t.contiguous() for t in (q[:, a], k[:, b], v[:, b])))
        assert torch.isfinite(o1).all() and torch.equal(o[:, a], o1) and torch.equal(lse[a], lse1), h
        if h in (0, Hkv - 1):
            heads = q[:, a].contiguous()
            ref = _oracle(heads.view(torch.int16).cpu().numpy().view(np.uint16), kb[:, b], vb[:, b], dob[:, a], L, K,
                          pe.Shape(L, K, n, 1, D).scale)
            assert rel_l2(bf16_to_f64(o1), ref["O"]) <= FWD_REL, h
            assert max_abs(lse1.double().cpu().numpy(), ref["LSE"]) <= LSE_ABS + 2e-6 * np.abs(ref["LSE"]).max(), h


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("form,seg,sets", [("dense", -1, 3), ("sampled", -1, 3), ("second_segment", 1, None), ("packed", -1, 3)])
def test_chunks_of_few_heads_in_a_backward_by_itself(form, seg, sets, D):
    """peagle_attn_bwd of four heads over a range of rows in chunks, with accumulate 0 and 1 on what the caller's tensors hold: the
    same bits with room for one set of partials (a launch and a sum for each chunk), and with accumulate what they held added."""
    from peagle_inputs import cod_depth_counts
    print(f"case chunks in a backward {form} D={D}", flush=True)
    Hq, Hkv, K = 4, 1, {"dense": 32, "packed": 16}.get(form, 7)
    if form == "dense":
        L, tm = 252, pe.peagle_build_tilemap(252, K, None, device=0)
    elif form == "packed":
        lens = [20, 290, 3, 41]
        L, tm = sum(lens), pe.peagle_build_tilemap_packed(lens, K, device=0)
    else:
        L, bounds = 1050, [0, 400, 1050] if seg >= 0 else None
        tm = pe.peagle_build_tilemap_sampled(cod_depth_counts(L, K, 0.9, 385), K, bounds, device=0)
    shape, T = pe.Shape(L, K, Hq, Hkv, D), tm.tokens(L)
    part, rest = 2 * Hq * ((L + 63) // 64 * 64) * D * 4, 2 * ((T * Hq * 4 + 255) // 256 * 256)
    need = pe.peagle_workspace_bytes(tm, shape)
    assert need == rest + (sets or (4 if D == 64 else 3)) * part
    g = torch.Generator(device="cuda").manual_seed(386)
    q, k, v, d_o = (torch.randn(T, H, D, generator=g, device="cuda").to(torch.bfloat16) for H in (Hq, Hkv, Hkv, Hq))
    old = [torch.randn(T, Hkv, D, generator=g, device="cuda") for _ in range(2)]
    o, lse = torch.zeros_like(q), torch.zeros((Hq, T), device="cuda")
    pe.peagle_attn_fwd(tm, shape, seg, q, k, v, o, lse)

    def results(n_bytes, accumulate):
        ws = torch.full((n_bytes,), 255, dtype=torch.uint8, device="cuda")  # (NaN)
        out = [torch.zeros_like(q), *(t.clone() for t in old)]
        pe.peagle_attn_bwd(tm, shape, seg, q, k, v, o, d_o, lse, *out, accumulate, ws)
        torch.cuda.synchronize()
        return out
    plain, added = results(need, 0), results(need, 1)
    for accumulate, got in ((0, plain), (1, added)):
        for a, b in zip(got, results(rest + part, accumulate)):
            assert torch.isfinite(a).all() and torch.equal(a, b), accumulate
    assert torch.equal(plain[0], added[0])
    for a, b, t in zip(added[1:], plain[1:], old):
        # (three chunks added to the tensor, three to each other, two subtractions: eight roundings of sums that are at most
        # twice what the result and the tensor are; keys that no row of the call sees are left as they were)
        seen = (b != t).any(dim=2).any(dim=1)
        assert seen.any() and (seg < 0) <= bool(seen.all())
        assert torch.equal(a[~seen], t[~seen])
        assert (a - b - t)[seen].abs().max() <= 16 * 2.0 ** -24 * float(b.abs().max() + t.abs().max())
