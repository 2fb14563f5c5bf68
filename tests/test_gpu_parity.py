"""HIP path vs CPU oracle, element by element, on identical seeded inputs.

Bars: expert indices, evicted slots, appended rows: bit-exact.  Attention output:
|d| <= 2e-3 + 1e-2 |ref| (bf16 storage, fp32 accumulate) plus a relative-L2 bound of 1e-3;
utilities: rel 1e-4.  Sizes span several tiles, several splits and ragged tails.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import pikv_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2508_06526_amd as pk  # noqa: E402
from gpu_harness import (DEV, DeviceCase, assert_utility_close, ensure_route_margin, t2n,  # noqa: E402
                         y_tolerance_ok)


def oracle_step(case, idx, gates, combine, utility=None, decay=1.0, scale=0.0):
    g = case.geo
    return orc.attend(case.q, case.K_shards, case.V_shards, case.n_valid, idx, gates, Hkv=g.Hkv,
                      E=g.E, S=g.S, dtype=g.dtype, rank=g.rank, U_K=case.U_K, U_V=case.U_V,
                      combine=combine, scale=scale, utility=utility, decay=decay, want_prob=True)


# ---------------------------------------------------------------------- route
ROUTE_CASES = [
    # (rows-shape geometry, k)
    dict(B=1, Hq=4, Hkv=4, D=64, E=4, S=8, k=2, dtype="f32", per_head_routing=True),
    dict(B=8, Hq=32, Hkv=32, D=128, E=16, S=8, k=2, dtype="bf16"),
    dict(B=1, Hq=32, Hkv=8, D=128, E=16, S=8, k=4, dtype="bf16"),
    dict(B=32, Hq=32, Hkv=32, D=128, E=8, S=8, k=2, dtype="bf16"),
    dict(B=3, Hq=2, Hkv=1, D=16, E=5, S=8, k=3, dtype="f32"),
    dict(B=5, Hq=4, Hkv=4, D=32, E=64, S=8, k=7, dtype="bf16"),
    dict(B=2, Hq=8, Hkv=8, D=64, E=1, S=8, k=1, dtype="bf16"),
    dict(B=4, Hq=8, Hkv=8, D=64, E=33, S=8, k=33, dtype="f32"),
]


@pytest.mark.parametrize("spec", ROUTE_CASES, ids=lambda s: "E%d_k%d_%s_B%d" % (s["E"], s["k"], s["dtype"], s["B"]))
@pytest.mark.parametrize("with_bias", [False, True])
def test_route_matches_oracle(spec, with_bias):
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=3, w_sigma=1.0 if g.dtype == "f32" else 0.02,
                             zipf_s=1.1 if with_bias else 0.0)
    ensure_route_margin(case, g.k)
    dc = DeviceCase(case)
    dc.route()
    x = np.ascontiguousarray(case.q.reshape(g.route_rows, g.d_r))
    idx, gates, probs = orc.route(x, case.W_r, g.k, bias=case.bias, dtype=g.dtype)
    np.testing.assert_array_equal(t2n(dc.topk), idx)
    np.testing.assert_allclose(t2n(dc.gates), gates, rtol=2e-5, atol=1e-7)
    np.testing.assert_allclose(t2n(dc.probs), probs, rtol=2e-5, atol=1e-7)


@pytest.mark.parametrize("rows", [257, 511, 513, 1027, 2051, 3000, 4096, 4099])
@pytest.mark.parametrize("E,dtype", [(8, "bf16"), (16, "bf16"), (24, "bf16"), (32, "bf16"), (36, "bf16"), (64, "bf16"), (4, "f32"),
                                     (8, "f32"), (16, "f32"), (64, "f32"), (6, "bf16"), (6, "f32"), (13, "f32"), (63, "f32")])
def test_route_of_many_rows_gives_each_row_its_own_bits(rows, E, dtype):
    """A prompt's rows share a block's pass over W_r, ceil(rows / 256) of them up to 16 in bf16, 2, 4 or 8 in fp32 or up
    to 16 in chunks of W_r, the last block partly filled; selection, gates and probabilities of a row are those
    of a call with few rows, bit for bit - every layout of the experts, with NaN and infinite logits among them."""
    k, d_r = 3, 520
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + E)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((rows, d_r), device=DEV, generator=gen)
    x[5, 7], x[rows - 1, 0], x[9] = float("nan"), float("inf"), 0.0
    x = x.to(tdt)
    W = (torch.randn((d_r, E), device=DEV, generator=gen) * 0.1).to(tdt)
    bias = torch.randn(E, device=DEV, generator=gen)

    def route(xs):
        n = xs.shape[0]
        out = (torch.full((n, k), -1, device=DEV, dtype=torch.int32), torch.zeros((n, k), device=DEV),
               torch.zeros((n, E), device=DEV))
        pk.pikv_route(xs, W, bias, n, d_r, E, k, *out)
        return [t2n(t) for t in out]

    whole = route(x)
    parts = [route(x[i:i + 200].contiguous()) for i in range(0, rows, 200)]
    for w, p in zip(whole, zip(*parts)):
        np.testing.assert_array_equal(w, np.concatenate(p))


@pytest.mark.parametrize("d_r", [1, 31, 127, 128, 130, 2048, 4104])
@pytest.mark.parametrize("E,dtype", [(1, "bf16"), (2, "bf16"), (5, "bf16"), (8, "bf16"), (10, "bf16"), (16, "bf16"), (24, "bf16"),
                                     (32, "bf16"), (33, "bf16"), (36, "bf16"), (62, "bf16"), (64, "bf16"),
                                     (1, "f32"), (3, "f32"), (6, "f32"), (12, "f32"), (40, "f32"), (63, "f32"), (4, "f32"), (8, "f32"),
                                     (16, "f32"), (64, "f32")])
def test_route_forms_agree_and_stay_within_their_rounding(E, dtype, d_r):
    """Whole and partial units of the contraction, every layout of the experts, rows in columns of their own or
    traded, words or single elements (x or W_r off by one element): the same bits, and within the rounding of
    the sums - at most a chain of d_r / 512 + 32 fp32 additions, exp to 4e-6 - of 64 bits."""
    k, rows = min(2, E), 1100
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1000 * E + d_r)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def at_offset(t, off):               # the same values, `off` elements into their buffer
        buf = torch.empty(t.numel() + off, device=DEV, dtype=t.dtype)
        buf[off:].copy_(t.reshape(-1))
        return buf[off:].view(t.shape)

    x = torch.randn((rows, d_r), device=DEV, generator=gen).to(tdt)
    W = (torch.randn((d_r, E), device=DEV, generator=gen) * d_r ** -0.5).to(tdt)

    def route(xs, Ws):
        n = xs.shape[0]
        out = (torch.full((n, k), -1, device=DEV, dtype=torch.int32), torch.zeros((n, k), device=DEV),
               torch.zeros((n, E), device=DEV))
        pk.pikv_route(xs, Ws, None, n, d_r, E, k, *out)
        return [t2n(t) for t in out]

    whole = route(x, W)
    logits = x.double() @ W.double()
    bound = (d_r / 512 + 32) * 2.0 ** -24 * (x.double().abs() @ W.double().abs())
    ref = torch.softmax(logits, 1)

    def assert_close(probs):
        assert ((torch.from_numpy(probs).to(DEV) - ref).abs() <= ref * (2 * bound.amax(1, keepdim=True) + 4e-6)).all()

    def assert_same(whole, variants):
        for xs, Ws in variants:
            for w, p in zip(whole, route(xs, Ws)):
                np.testing.assert_array_equal(w[:xs.shape[0]], p)

    assert_close(whole[2])
    moved = at_offset(W, 1)
    assert_same(whole, [(x[:300].contiguous(), W), (x[:3].contiguous(), W), (at_offset(x[:3], 1), W), (at_offset(x[:700], 1), W)])
    if dtype == "f32" and E in (4, 8, 16, 32, 64):           # rows of W_r that are whole chunks lose their layout
        whole = route(x, moved)
        assert_close(whole[2])
    assert_same(whole, [(x[:3].contiguous(), moved), (x[:300].contiguous(), moved), (x, moved)])


@pytest.mark.parametrize("E,d_r", [(3, 9000), (6, 750), (6, 751), (13, 512), (13, 513), (12, 256), (12, 257), (63, 128), (63, 129)])
def test_route_forms_on_both_sides_of_the_line_between_single_elements_and_chunks(E, d_r):
    test_route_forms_agree_and_stay_within_their_rounding(E, "f32", d_r)


def test_route_exact_ties_lower_index_first():
    rng = np.random.default_rng(6)
    rows, d_r = 64, 32
    x = rng.integers(-3, 4, size=(rows, d_r)).astype(np.float32)
    Wb = rng.integers(-2, 3, size=(d_r, 4)).astype(np.float32)
    W = np.ascontiguousarray(np.concatenate([Wb, Wb[:, [1, 3]], Wb[:, [0]], Wb], axis=1))   # E = 11
    x[0] = 0
    for dtype in ("f32", "bf16"):
        xs, Ws = wl.encode(x, dtype), wl.encode(W, dtype)
        for k in (1, 3, 6, 11):
            idx, gates, _ = orc.route(xs, Ws, k, dtype=dtype)
            from gpu_harness import dev_storage
            tk = torch.zeros((rows, k), device=DEV, dtype=torch.int32)
            tg = torch.zeros((rows, k), device=DEV)
            pk.pikv_route(dev_storage(xs, dtype), dev_storage(Ws, dtype), None, rows, d_r, 11, k, tk, tg)
            np.testing.assert_array_equal(t2n(tk), idx)
            np.testing.assert_allclose(t2n(tg), gates, rtol=2e-5)


def test_round_robin_router_matches_oracle_and_feeds_attention():
    g = wl.Geometry(B=5, Hq=4, Hkv=2, D=64, E=7, S=90, k=3, dtype="bf16")
    case = wl.make_host_case(g, seed=17, n_valid="ragged")
    dc = DeviceCase(case)
    for step in (0, 4, 123456789):
        pk.pikv_route_round_robin(g.B, g.E, g.k, step, dc.topk, dc.gates)
        idx, gates = orc.route_round_robin(g.B, g.E, g.k, step)
        np.testing.assert_array_equal(t2n(dc.topk), idx)
        np.testing.assert_array_equal(t2n(dc.gates), gates)
    ref = oracle_step(case, idx, gates, orc.COMBINE_LOCAL)
    dc.attend(combine=pk.COMBINE_LOCAL)
    ok, emax, l2 = y_tolerance_ok(t2n(dc.y), ref["y"], g.dtype)
    assert ok, (emax, l2)
    with pytest.raises(pk.PikvError):
        pk.pikv_route_round_robin(g.B, g.E, g.E + 1, 0, dc.topk, dc.gates)


# ------------------------------------------------------------------ attention
ATTN_CASES = {
    # config 1 itself: per-head routing, fp32
    "c1_tiny_f32": (dict(B=1, Hq=4, Hkv=4, D=64, E=4, S=256, k=2, dtype="f32", per_head_routing=True), "full"),
    # scaled config 2: G=1, bf16, several splits and a ragged tail
    "c2_scaled": (dict(B=2, Hq=4, Hkv=4, D=128, E=6, S=700, k=2, dtype="bf16"), "ragged"),
    # scaled config 3: GQA group of 4, k=4
    "c3_scaled": (dict(B=1, Hq=8, Hkv=2, D=128, E=8, S=1100, k=4, dtype="bf16"), "ragged"),
    "gqa2": (dict(B=2, Hq=4, Hkv=2, D=64, E=4, S=300, k=2, dtype="bf16"), "ragged"),
    "gqa8": (dict(B=1, Hq=8, Hkv=1, D=128, E=4, S=260, k=2, dtype="bf16"), "full"),
    "gqa3_generic": (dict(B=1, Hq=6, Hkv=2, D=64, E=4, S=150, k=3, dtype="bf16"), "ragged"),
    # matrix-core grouped-query kernel (bf16, D=128): odd group sizes, the 16-head limit, short tails
    "gqa3_d128": (dict(B=2, Hq=6, Hkv=2, D=128, E=4, S=333, k=2, dtype="bf16"), "ragged"),
    "gqa16_d128": (dict(B=1, Hq=16, Hkv=1, D=128, E=3, S=1500, k=2, dtype="bf16"), "ragged"),
    "gqa5_d128_tiny": (dict(B=1, Hq=5, Hkv=1, D=128, E=2, S=7, k=2, dtype="bf16"), "full"),
    # more than 16 rows per kv head: two and four 16-row tiles sharing every K/V load
    "gqa32_two_row_tiles": (dict(B=1, Hq=32, Hkv=1, D=128, E=2, S=70, k=1, dtype="bf16"), "full"),
    "gqa17_d128": (dict(B=2, Hq=34, Hkv=2, D=128, E=3, S=400, k=2, dtype="bf16"), "ragged"),
    "gqa48_d128": (dict(B=1, Hq=96, Hkv=2, D=128, E=3, S=700, k=2, dtype="bf16"), "ragged"),
    "gqa64_d128": (dict(B=1, Hq=128, Hkv=2, D=128, E=4, S=1300, k=3, dtype="bf16"), "ragged"),
    # scaled config 5: rank-32 codes
    "c5_scaled": (dict(B=2, Hq=4, Hkv=4, D=128, E=6, S=900, k=2, dtype="bf16", rank=32), "ragged"),
    "rank16_gqa4": (dict(B=1, Hq=8, Hkv=2, D=64, E=4, S=520, k=2, dtype="bf16", rank=16), "ragged"),
    "rank64_f32": (dict(B=1, Hq=2, Hkv=2, D=128, E=3, S=130, k=2, dtype="f32", rank=64), "full"),
    "f32_d128": (dict(B=1, Hq=2, Hkv=1, D=128, E=3, S=100, k=3, dtype="f32"), "ragged"),
    "d32_bf16": (dict(B=2, Hq=2, Hkv=2, D=32, E=4, S=515, k=2, dtype="bf16"), "ragged"),
    "d16_bf16_perhead": (dict(B=2, Hq=4, Hkv=2, D=16, E=4, S=1030, k=2, dtype="bf16", per_head_routing=True), "ragged"),
    "k_equals_E": (dict(B=1, Hq=4, Hkv=4, D=64, E=4, S=129, k=4, dtype="bf16"), "ragged"),
    "one_slot": (dict(B=1, Hq=2, Hkv=2, D=64, E=2, S=1, k=2, dtype="bf16"), "full"),
    # the limits: longest shards, most query heads, most experts
    "long_shard_70k": (dict(B=1, Hq=4, Hkv=2, D=128, E=2, S=70000, k=2, dtype="bf16"), "ragged"),
    "long_shard_g1_40k": (dict(B=1, Hq=2, Hkv=2, D=64, E=2, S=40000, k=1, dtype="bf16"), "full"),
    "hq256": (dict(B=1, Hq=256, Hkv=32, D=64, E=2, S=64, k=2, dtype="bf16"), "ragged"),
    "e64_k64": (dict(B=1, Hq=2, Hkv=2, D=32, E=64, S=40, k=64, dtype="bf16"), "ragged"),
    # the utility kernel's shape for hundreds of query rows: heads chosen per head (an expert's
    # active heads differ in number, down to none), slot tiles with a ragged end
    "hq160_perhead": (dict(B=2, Hq=160, Hkv=4, D=32, E=3, S=150, k=2, dtype="bf16", per_head_routing=True), "ragged"),
    "hq128_k1": (dict(B=1, Hq=128, Hkv=2, D=128, E=5, S=333, k=1, dtype="bf16"), "ragged"),
}


def random_selection(g, seed):
    rng = np.random.default_rng(seed)
    idx = np.stack([rng.permutation(g.E)[:g.k] for _ in range(g.route_rows)]).astype(np.int32)
    gates = rng.random((g.route_rows, g.k)).astype(np.float32) + 0.05
    gates /= gates.sum(-1, keepdims=True)
    return idx, gates.astype(np.float32)


@pytest.mark.parametrize("name", sorted(ATTN_CASES))
@pytest.mark.parametrize("combine", [orc.COMBINE_LSE, orc.COMBINE_LOCAL], ids=["lse", "local"])
@pytest.mark.parametrize("use_gates", [True, False], ids=["gates", "mask"])
def test_attention_and_utility_match_oracle(name, combine, use_gates):
    spec, nv = ATTN_CASES[name]
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=11, kv="lognormal_token", n_valid=nv, utility0="exp")
    idx, gates = random_selection(g, 5)
    if not use_gates:
        gates = None
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, gates, combine, utility=u_ref, decay=0.9)

    dc = DeviceCase(case)
    d_idx = torch.from_numpy(idx).to(DEV)
    d_gates = None if gates is None else torch.from_numpy(gates).to(DEV)
    dc.attend(topk=d_idx, gates=d_gates, combine=combine)
    dc.update_utility(0.9, topk=d_idx)

    y = t2n(dc.y)
    ok, emax, l2 = y_tolerance_ok(y, ref["y"], g.dtype)
    assert ok, "y mismatch: max abs %.3e, rel L2 %.3e" % (emax, l2)
    np.testing.assert_allclose(t2n(dc.row_max), ref["row_max"], rtol=1e-4, atol=1e-5)
    np.testing.assert_allclose(t2n(dc.row_norm), ref["row_norm"], rtol=1e-4, atol=1e-9)
    assert_utility_close(t2n(dc.utility), u_ref)
    # per-entry probabilities rebuilt from the emitted scores and (shift, coef)
    sc, co = t2n(dc.scores).astype(np.float64), t2n(dc.slot_coef).astype(np.float64)
    for b in range(g.B):
        for h in range(g.Hq):
            row = b * g.Hq + h if g.per_head_routing else b
            for j in range(g.k):
                n = case.n_valid[b, idx[row, j]]
                p = co[b, h, j, 1] * np.exp(sc[b, h, j, :n] - co[b, h, j, 0])
                np.testing.assert_allclose(p, ref["prob"][b, h, j, :n], rtol=1e-4, atol=1e-10)


@pytest.mark.parametrize("spec", [
    dict(B=2, Hq=16, Hkv=2, D=128, E=4, S=300, k=2, dtype="bf16", tq=4),      # 8 rows per kv head
    dict(B=1, Hq=64, Hkv=2, D=128, E=4, S=500, k=2, dtype="bf16", tq=8),      # 32 rows: two row tiles
    dict(B=2, Hq=128, Hkv=2, D=128, E=3, S=200, k=2, dtype="bf16", tq=16),    # 64 rows: four row tiles
    dict(B=1, Hq=72, Hkv=3, D=128, E=3, S=150, k=3, dtype="bf16", tq=6),      # 24 rows, three kv heads
], ids=["tq4", "tq8", "tq16", "tq6_kv3"])
@pytest.mark.parametrize("combine", [orc.COMBINE_LSE, orc.COMBINE_LOCAL], ids=["lse", "local"])
def test_multi_query_step_in_token_major_layout(spec, combine):
    """Draft queries of a multi-query step in their natural layout, q [B, tq, heads, D] with
    desc.tq = tq: routing by the tile's first query, attention of every (draft, head) row over the
    selected shards, outputs back in [B, tq, heads] order, utilities summed over all rows.  The
    oracle sees the same rows as Hq = tq * heads plain query heads in kv-head-first order."""
    from gpu_harness import dev_storage
    g = wl.Geometry(token_major=True, **spec)
    case = wl.make_host_case(g, seed=71, n_valid="ragged", utility0="exp", w_sigma=0.02)
    perm = wl.token_major_rows(g.Hq, g.Hkv, g.tq)           # internal row -> caller row
    q_caller = np.empty_like(case.q)
    q_caller[:, perm] = case.q                               # the caller's [B, tq*heads, D]
    # the router sees the caller's flat vector
    probe = case.clone()
    probe.q = q_caller
    ensure_route_margin(probe, g.k)
    q_caller = probe.q
    case.q = np.ascontiguousarray(q_caller[:, perm])        # oracle order of the same rows
    dc = DeviceCase(case)
    dc.q = dev_storage(q_caller, g.dtype)
    dc.desc = pk.make_desc(g.B, g.Hq, g.Hkv, g.D, g.E, g.S, dtype=pk.binding.BF16, stride_h=dc.stride_h,
                           stride_s=dc.stride_s, tq=g.tq)
    dc.route()
    x = np.ascontiguousarray(wl.routing_rows(g, q_caller))   # the tile's first query routes the step
    assert x.shape == (g.B, g.Hq // g.tq * g.D)
    np.testing.assert_array_equal(x, q_caller[:, :g.Hq // g.tq].reshape(g.B, -1))
    idx, gates, _ = orc.route(x, case.W_r, g.k, dtype=g.dtype)
    np.testing.assert_array_equal(t2n(dc.topk), idx)
    dc.attend(combine=combine)
    dc.update_utility(0.9)
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, t2n(dc.gates), combine, utility=u_ref, decay=0.9)
    y = t2n(dc.y)[:, perm]                                   # back to the oracle's row order
    ok, emax, l2 = y_tolerance_ok(y, ref["y"], g.dtype)
    assert ok, (emax, l2)
    np.testing.assert_allclose(t2n(dc.row_max)[:, perm], ref["row_max"], rtol=1e-4, atol=1e-5)
    np.testing.assert_allclose(t2n(dc.row_norm)[:, perm], ref["row_norm"], rtol=1e-4, atol=1e-9)
    assert_utility_close(t2n(dc.utility), u_ref)


@pytest.mark.parametrize("spec", [
    dict(B=2, Hq=34, Hkv=2, D=128, E=3, S=200, k=2, dtype="bf16", tq=17),     # one head per draft; a second row tile of one row
    dict(B=1, Hq=45, Hkv=3, D=128, E=4, S=700, k=4, dtype="bf16", tq=5),      # three heads per draft, 15 rows, empty splits
    dict(B=1, Hq=99, Hkv=3, D=128, E=3, S=257, k=2, dtype="bf16", tq=3),      # 33 rows: the third row tile of one row
], ids=["tq17_g1", "tq5_g3", "tq3_g11"])
def test_draft_rows_of_odd_groups(spec):
    """The caller's rows of a group (the quotient by the heads of a draft) and the merge of a block's waves, four
    values per thread, at row tiles that end in one row."""
    test_multi_query_step_in_token_major_layout(spec, orc.COMBINE_LSE)


def test_library_opened_before_torch_still_launches():
    """A caller may load the binding's library before it ever imports torch; both must end up on
    one HIP runtime (a kernel launched through a second copy fails on torch's streams).  Runs in
    a fresh interpreter, because this process has imported torch long ago."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = (
        "import sys; sys.path.insert(0, %r)\n"
        "import paper_2508_06526_amd as pk\n"
        "assert pk.load_library().pikv_version() >= 300\n"
        "import torch\n"
        "x = torch.eye(8, device='cuda:0'); W = torch.eye(8, device='cuda:0')\n"
        "idx = torch.zeros((8, 1), device='cuda:0', dtype=torch.int32); g = torch.zeros((8, 1), device='cuda:0')\n"
        "pk.pikv_route(x, W, None, 8, 8, 8, 1, idx, g)\n"
        "torch.cuda.synchronize()\n"
        "assert idx.flatten().tolist() == list(range(8)), idx\n"
        "print('ok')\n" % root)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "ok" in r.stdout, (r.stdout[-500:], r.stderr[-1500:])


def test_multi_query_layout_is_refused_where_no_kernel_takes_it():
    fake = torch.zeros(64, device=DEV)
    for kw in (dict(D=64), dict(rank=32), dict(dtype=pk.binding.F32)):     # only bf16 rows of 128 values
        args = dict(D=128, rank=0, dtype=pk.binding.BF16)
        args.update(kw)
        desc = pk.make_desc(1, 16, 2, args["D"], 4, 64, rank=args["rank"], dtype=args["dtype"], tq=4)
        ws = torch.empty(1 << 20, device=DEV, dtype=torch.uint8)
        with pytest.raises(pk.PikvError) as err:
            pk.pikv_sharded_attn(desc, fake, fake, fake, fake, fake, fake, fake, None, 2, pk.COMBINE_LSE, 0.0,
                                 fake, None, None, None, None, ws)
        assert err.value.status == -2


def random_geometry(rng):
    D = int(rng.choice([16, 32, 64, 128]))
    dtype = str(rng.choice(["bf16", "bf16", "f32"]))
    rank = int(rng.choice([0, 0, 16, 32, 64]))
    if rank >= D:
        rank = 0
    Hkv = int(rng.choice([1, 2, 3, 4]))
    G = int(rng.choice([1, 1, 2, 3, 4, 5, 8, 16, 24, 40]))
    E = int(rng.integers(1, 10))
    k = int(rng.integers(1, E + 1))
    per_head = bool(rng.random() < 0.25)
    return dict(B=int(rng.integers(1, 4)), Hq=Hkv * G, Hkv=Hkv, D=D, E=E, S=int(rng.integers(1, 700)), k=k,
                dtype=dtype, rank=rank, per_head_routing=per_head)


@pytest.mark.parametrize("seed", range(24))
def test_attention_on_random_geometries(seed):
    """Seeded sweep over shapes nobody hand-picked: head grouping, widths, code ranks, shard counts,
    ragged fills, both combine modes, gates or mask, split counts forced or chosen."""
    rng = np.random.default_rng(1000 + seed)
    g = wl.Geometry(**random_geometry(rng))
    case = wl.make_host_case(g, seed=seed, kv="lognormal_token", n_valid=str(rng.choice(["ragged", "full"])),
                             utility0="exp")
    idx, gates = random_selection(g, 50 + seed)
    if rng.random() < 0.3:
        gates = None
    combine = int(rng.choice([orc.COMBINE_LSE, orc.COMBINE_LOCAL]))
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, gates, combine, utility=u_ref, decay=0.7)
    forced = int(rng.choice([0, 0, 1, 3, 7]))
    pk.pikv_set_attn_split(forced)
    try:
        dc = DeviceCase(case)
        d_idx = torch.from_numpy(idx).to(DEV)
        d_gates = None if gates is None else torch.from_numpy(gates).to(DEV)
        dc.attend(topk=d_idx, gates=d_gates, combine=combine)
        dc.update_utility(0.7, topk=d_idx)
        y, u = t2n(dc.y), t2n(dc.utility)
    finally:
        pk.pikv_set_attn_split(0)
    ok, emax, l2 = y_tolerance_ok(y, ref["y"], g.dtype)
    assert ok, "geometry %s: max abs %.3e, rel L2 %.3e" % (g, emax, l2)
    np.testing.assert_allclose(t2n(dc.row_max), ref["row_max"], rtol=1e-4, atol=1e-5)
    assert_utility_close(u, u_ref)


# Groups of query heads on the matrix cores at every row width: edges of the 16-row tiles and of the
# 32-, 64- and 128-row entry tiles, shards shorter than one of them, odd capacities (score rows that
# are no whole 16-byte chunks), every decoder width, and a query that is not 16-byte aligned.
GROUPED_ROWS = [
    dict(B=2, Hq=4, Hkv=2, D=16, E=3, S=127, k=2), dict(B=1, Hq=33, Hkv=1, D=16, E=2, S=516, k=2),
    dict(B=1, Hq=9, Hkv=3, D=32, E=3, S=65, k=2), dict(B=1, Hq=34, Hkv=2, D=32, E=2, S=257, k=1),
    dict(B=1, Hq=64, Hkv=1, D=32, E=2, S=31, k=2), dict(B=2, Hq=14, Hkv=2, D=64, E=3, S=63, k=2),
    dict(B=1, Hq=32, Hkv=2, D=64, E=2, S=1028, k=2), dict(B=1, Hq=17, Hkv=1, D=64, E=2, S=515, k=1),
    dict(B=1, Hq=128, Hkv=2, D=64, E=2, S=300, k=2), dict(B=1, Hq=6, Hkv=2, D=128, E=2, S=33, k=2),
    dict(B=1, Hq=4, Hkv=2, D=128, E=3, S=129, k=2, rank=16), dict(B=1, Hq=36, Hkv=1, D=16, E=2, S=130, k=2, rank=16),
    dict(B=2, Hq=10, Hkv=2, D=64, E=3, S=511, k=3, rank=32), dict(B=1, Hq=34, Hkv=2, D=128, E=2, S=66, k=1, rank=32),
    dict(B=1, Hq=6, Hkv=2, D=16, E=2, S=64, k=2, rank=32), dict(B=1, Hq=7, Hkv=1, D=128, E=3, S=1001, k=2, rank=64),
    dict(B=1, Hq=20, Hkv=1, D=32, E=2, S=200, k=2, rank=64), dict(B=1, Hq=40, Hkv=1, D=128, E=2, S=95, k=2, rank=64),
]


@pytest.mark.parametrize("spec", GROUPED_ROWS, ids=lambda s: "D%d_r%d_G%d_S%d" % (s["D"], s.get("rank", 0), s["Hq"] // s["Hkv"], s["S"]))
@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "q_off_by_one"])
def test_grouped_rows_of_every_width_match_oracle(spec, offset):
    """y against the fp64 oracle: exact products and fp32 sums, 2.5e-7 measured for rows and codes narrower
    than 128 values (with probabilities of a part less, 2.3e-6) - and for rows of 128 values
    probabilities of 17 bits (2e-6 measured).  Small calls, which the one-head kernel takes in part."""
    g = wl.Geometry(dtype="bf16", **spec)
    case = wl.make_host_case(g, seed=g.S + g.Hq, kv="lognormal_token", n_valid="ragged", utility0="exp")
    idx, gates = random_selection(g, g.S)
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE, utility=u_ref, decay=0.9)
    dc = DeviceCase(case)
    shifted = torch.empty(dc.q.numel() + offset, device=DEV, dtype=dc.q.dtype)
    shifted[offset:] = dc.q.flatten()
    dc.q = shifted[offset:].view(g.B, g.Hq, g.D)
    d_idx, d_gates = torch.from_numpy(idx).to(DEV), torch.from_numpy(gates).to(DEV)
    dc.attend(topk=d_idx, gates=d_gates)
    dc.update_utility(0.9, topk=d_idx)
    y = t2n(dc.y)
    assert np.linalg.norm(y - ref["y"]) <= (8e-6 if g.width == 128 else 1e-6) * np.linalg.norm(ref["y"])
    np.testing.assert_allclose(t2n(dc.row_max), ref["row_max"], rtol=1e-5, atol=1e-6)
    assert_utility_close(t2n(dc.utility), u_ref)
    with_scores = y
    dc.attend(topk=d_idx, gates=d_gates, want_scores=False)     # the kernel without score output: the same bits
    np.testing.assert_array_equal(t2n(dc.y), with_scores)


def check_group(case, want_rel, forced=0):
    """Attention (with scores) and utility of one call against the fp64 oracle."""
    g = case.geo
    idx, gates = random_selection(g, g.S)
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE, utility=u_ref, decay=0.9)
    d_idx, d_gates = torch.from_numpy(idx).to(DEV), torch.from_numpy(gates).to(DEV)
    for split in (forced if isinstance(forced, tuple) else (forced,)):
        pk.pikv_set_attn_split(split)
        try:
            d = DeviceCase(case)
            d.attend(topk=d_idx, gates=d_gates)
            d.update_utility(0.9, topk=d_idx)
            y, sc = t2n(d.y), t2n(d.scores)
        finally:
            pk.pikv_set_attn_split(0)
        assert np.linalg.norm(y - ref["y"]) <= want_rel * np.linalg.norm(ref["y"])
        assert_utility_close(t2n(d.utility), u_ref)
        n = np.take_along_axis(case.n_valid, idx, axis=1)                       # [B, k]
        live = np.broadcast_to((np.arange(g.S) < n[:, :, None])[:, None], sc.shape)
        assert np.isfinite(sc[live]).all() and np.isnan(sc[~live]).all()       # written up to the count, not past it


@pytest.mark.parametrize("D,rank", [(16, 0), (32, 0), (64, 0), (128, 16), (64, 32), (128, 64)], ids=lambda v: str(v))
@pytest.mark.parametrize("G", [16, 31, 64])
@pytest.mark.parametrize("S", [1100, 1103])
def test_groups_on_the_matrix_cores_in_both_forms_of_the_score_output(D, rank, G, S):
    """100 units, more than the one-head kernel is given.  In one split the scores of a block (70 KB at 16 rows)
    do not fit the LDS and are written from the loop, in sixteen they are staged; whole and
    ragged counts, score rows that are whole 16-byte chunks and not, all row tiles, widths and decoders.
    y: 3-part probabilities and fp32 sums, 2.5e-7 measured (a part less gives 2.3e-6)."""
    g = wl.Geometry(B=25, Hq=G, Hkv=1, D=D, rank=rank, E=4, S=S, k=4, dtype="bf16")
    case = wl.make_host_case(g, seed=S + G, n_valid="ragged", utility0="exp")
    case.n_valid[0] = [S, S - 1, 1, 129]
    check_group(case, 1e-6, forced=(1, 16))


@pytest.mark.parametrize("spec,most", [(dict(Hq=64, D=64), 2.1e-7), (dict(Hq=16, D=64), 2.1e-7), (dict(Hq=32, D=128, rank=32), 2.35e-7),
                                       (dict(Hq=32, D=128, rank=16), 2.4e-7), (dict(Hq=64, D=128, rank=64), 2.7e-7),
                                       (dict(Hq=32, D=128, S=5000), 1e-6), (dict(Hq=64, D=128, S=5000), 1e-6)],
                         ids=lambda v: "" if isinstance(v, float) else "D%d_r%d_G%d" % (v["D"], v.get("rank", 0), v["Hq"] // 8))
def test_long_blocks_of_groups_keep_the_precision_of_short_ones(spec, most):
    """48 units: blocks of up to 512 KiB, in which a wave adds 8 tiles to its running sums.  Error of y with the products of
    a tile summed apart 1.78, 1.73, 2.09, 2.18 and 2.41e-7 (short blocks 1.76, 1.77, 2.03, 2.26, 2.47), with products that
    accumulate 2.52, 2.45, 2.64, 2.72 and 2.98; rows of 128 values 2.0e-7 with probabilities of three
    parts, 2.0e-6 with two (short blocks 1.83e-6).  The bounds lie between."""
    g = wl.Geometry(**dict(dict(B=2, Hkv=8, E=3, S=8192, k=3, dtype="bf16"), **spec))
    case = wl.make_host_case(g, seed=1, utility0="exp")
    check_group(case, most)
    idx, gates = (torch.from_numpy(a).to(DEV) for a in random_selection(g, g.S))
    y = []
    for want_scores in (True, False):
        d = DeviceCase(case)
        d.attend(topk=idx, gates=gates, want_scores=want_scores)
        y.append(t2n(d.y))
    np.testing.assert_array_equal(*y)


@pytest.mark.parametrize("spec", [
    # either side of: 48, 64 and 96 blocks, the bytes re-read, and 28 MB of K/V for two heads over 16 values
    dict(B=24, Hq=48, Hkv=2, D=64, S=300, k=1), dict(B=49, Hq=24, Hkv=1, D=64, S=300, k=1),
    dict(B=32, Hq=10, Hkv=2, D=32, S=257, k=1), dict(B=13, Hq=5, Hkv=1, D=32, S=257, k=5),
    dict(B=24, Hq=12, Hkv=4, D=128, rank=16, S=130, k=1), dict(B=97, Hq=3, Hkv=1, D=16, S=130, k=1),
    dict(B=2, Hq=24, Hkv=2, D=64, S=5461, k=2), dict(B=2, Hq=24, Hkv=2, D=64, S=5463, k=2),
    dict(B=8, Hq=16, Hkv=8, D=16, S=3417, k=2), dict(B=8, Hq=16, Hkv=8, D=16, S=3418, k=2),
    dict(B=4, Hq=18, Hkv=6, D=64, rank=64, S=128, k=4), dict(B=4, Hq=18, Hkv=6, D=64, rank=64, S=129, k=4),
    dict(B=64, Hq=64, Hkv=16, D=32, S=1300, k=1),       # finer splits, so that the scores fit the LDS
], ids=lambda s: "B%d_G%d_D%d_r%d_S%d" % (s["B"], s["Hq"] // s["Hkv"], s["D"], s.get("rank", 0), s["S"]))
def test_narrow_groups_on_both_sides_of_the_choice_of_kernel(spec):
    """One head per block of the plain kernel, or whole groups on the matrix cores: the same result."""
    g = wl.Geometry(E=spec["k"], dtype="bf16", **spec)
    check_group(wl.make_host_case(g, seed=g.S, n_valid="ragged", utility0="exp"), 1e-6)


@pytest.mark.parametrize("spec", [
    dict(B=1, Hq=6, Hkv=2, D=16, E=2, S=1024, k=2), dict(B=1, Hq=16, Hkv=2, D=32, E=2, S=1024, k=2),
    dict(B=16, Hq=14, Hkv=2, D=64, E=4, S=1024, k=4), dict(B=8, Hq=48, Hkv=2, D=64, E=4, S=1024, k=4),
    dict(B=2, Hq=128, Hkv=2, D=64, E=4, S=4096, k=4), dict(B=4, Hq=16, Hkv=4, D=128, E=4, S=1024, k=4, rank=16),
    dict(B=8, Hq=20, Hkv=2, D=64, E=4, S=1024, k=4, rank=32), dict(B=4, Hq=32, Hkv=4, D=128, E=2, S=2048, k=2, rank=64),
    dict(B=8, Hq=64, Hkv=1, D=32, E=4, S=4096, k=4, rank=32),
], ids=lambda s: "D%d_r%d_G%d" % (s["D"], s.get("rank", 0), s["Hq"] // s["Hkv"]))
def test_infinite_entries_of_narrow_groups_stay_infinite(spec):
    """A value of +-Inf with a probability above zero makes its output +-Inf (not NaN: the probability's
    bf16 parts must not meet it with a zero or a negative one), and an entry whose code is infinite so that it
    scores -Inf drops out of the softmax; what neither reaches keeps its tolerance."""
    g = wl.Geometry(dtype="bf16", **spec)
    case = wl.make_host_case(g, seed=g.S + g.Hq, utility0="exp")
    inf, ninf = np.uint16(0x7F80), np.uint16(0xFF80)
    for s, at in ((0, 700), (g.B * g.E - 1, g.S - 300)):      # shards are [Hkv, S, width]
        case.V_shards[s][0, at, 3], case.V_shards[s][g.Hkv - 1, at + 1, 5] = inf, ninf
        if g.rank:     # q and the decoder row of one code column are positive: the entry scores -Inf for all heads
            case.K_shards[s][0, at + 9, 7] = ninf
            case.V_shards[s][0, at + 9] = 0
    if g.rank:
        case.q &= np.uint16(0x7FFF)
        case.U_K[:, 7] &= np.uint16(0x7FFF)
    idx, gates = random_selection(g, 2)
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE)
    dc = DeviceCase(case)
    d_idx, d_gates = torch.from_numpy(idx).to(DEV), torch.from_numpy(gates).to(DEV)
    for want_scores in (True, False):
        dc.y.fill_(7.0)
        dc.attend(topk=d_idx, gates=d_gates, want_scores=want_scores)
        y = t2n(dc.y)
        assert np.isinf(ref["y"]).any() and np.isfinite(ref["y"]).any()
        for kind in (np.isposinf, np.isneginf, np.isnan):
            np.testing.assert_array_equal(kind(y), kind(ref["y"]), err_msg=kind.__name__)
        ok = np.isfinite(ref["y"])
        assert np.linalg.norm(y[ok] - ref["y"][ok]) <= 1e-6 * np.linalg.norm(ref["y"][ok])


@pytest.mark.parametrize("spec", [
    dict(B=2, Hq=6, Hkv=2, D=128, S=17), dict(B=1, Hq=10, Hkv=2, D=128, S=1030), dict(B=2, Hq=32, Hkv=2, D=128, S=513),
    # groups of four: the plain kernel's
    dict(B=1, Hq=8, Hkv=2, D=128, S=1030), dict(B=2, Hq=8, Hkv=2, D=64, S=1), dict(B=1, Hq=16, Hkv=4, D=16, rank=16, S=130),
    dict(B=1, Hq=64, Hkv=2, D=128, S=300),                      # 32 heads in two blocks of 16
    dict(B=1, Hq=36, Hkv=2, D=64, S=700), dict(B=3, Hq=10, Hkv=2, D=64, S=129), dict(B=1, Hq=34, Hkv=2, D=64, S=90),
    dict(B=2, Hq=14, Hkv=2, D=32, S=1025), dict(B=1, Hq=16, Hkv=1, D=16, S=1999), dict(B=2, Hq=6, Hkv=2, D=64, S=1),
    dict(B=1, Hq=16, Hkv=2, D=32, S=5000),                      # scores that fit the LDS in finer splits only
    dict(B=2, Hq=12, Hkv=4, D=64, rank=16, S=260), dict(B=1, Hq=30, Hkv=2, D=128, rank=32, S=515),
    dict(B=2, Hq=16, Hkv=2, D=32, rank=64, S=300), dict(B=1, Hq=24, Hkv=4, D=16, rank=16, S=130),
    dict(B=1, Hq=16, Hkv=1, D=128, rank=64, S=1100),
], ids=lambda s: "D%d_r%d_G%d_S%d" % (s["D"], s.get("rank", 0), s["Hq"] // s["Hkv"], s["S"]))
def test_groups_of_fp32_rows_match_oracle(spec):
    """Groups of 3 and of 5 and more heads on the fp32 matrix cores: tiles of 16 to 64 entries and their remainders, scores
    staged, in finer splits and written from the loop, groups that no number of heads up to 16 but one divides.
    fp32 sums, 1.7e-7 measured."""
    g = wl.Geometry(E=3, k=2, dtype="f32", **spec)
    case = wl.make_host_case(g, seed=g.S, n_valid="ragged", utility0="exp")
    case.n_valid[0] = [g.S, max(1, g.S - 1), (g.S + 1) // 2]
    check_group(case, 1e-6, forced=(0, 1, 7))


@pytest.mark.parametrize("spec", [dict(B=2, Hq=16, Hkv=2, D=128), dict(B=2, Hq=12, Hkv=2, D=64), dict(B=1, Hq=32, Hkv=2, D=16),
                                  dict(B=2, Hq=16, Hkv=2, D=64, rank=32), dict(B=2, Hq=8, Hkv=2, D=64, rank=32)],
                         ids=lambda s: "D%d_r%d_G%d" % (s["D"], s.get("rank", 0), s["Hq"] // s["Hkv"]))
def test_infinite_entries_of_fp32_groups_stay_infinite(spec):
    g = wl.Geometry(E=2, k=2, S=512, dtype="f32", **spec)
    case = wl.make_host_case(g, seed=g.Hq, utility0="exp")
    for s, at in ((0, 300), (g.B * g.E - 1, 100)):
        case.V_shards[s][0, at, 3], case.V_shards[s][g.Hkv - 1, at + 1, 5] = np.inf, -np.inf
    idx, gates = random_selection(g, 2)
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE)
    dc = DeviceCase(case)
    dc.attend(topk=torch.from_numpy(idx).to(DEV), gates=torch.from_numpy(gates).to(DEV))
    y = t2n(dc.y)
    assert np.isinf(ref["y"]).any()
    for kind in (np.isposinf, np.isneginf, np.isnan):
        np.testing.assert_array_equal(kind(y), kind(ref["y"]), err_msg=kind.__name__)
    ok = np.isfinite(ref["y"])
    assert np.linalg.norm(y[ok] - ref["y"][ok]) <= 1e-6 * np.linalg.norm(ref["y"][ok])


@pytest.mark.parametrize("spec", [dict(Hq=16, D=128, S=17), dict(Hq=6, D=64, S=33), dict(Hq=16, D=32, S=65), dict(Hq=12, D=16, S=200),
                                  dict(Hq=16, D=64, S=41, rank=32)],
                         ids=lambda s: "D%d_r%d_G%d" % (s["D"], s.get("rank", 0), s["Hq"] // 2))
def test_infinities_in_the_last_entry_of_fp32_groups(spec):
    """A shard's last tile is partly past its entries, and may be its wave's first: an infinite value in the last entry
    is no NaN of the rows behind it, and a last entry that scores -Inf drops out of the softmax."""
    g = wl.Geometry(B=1, Hkv=2, E=2, k=2, dtype="f32", **spec)
    idx, gates = random_selection(g, 2)
    for kind in ("value", "score"):
        case = wl.make_host_case(g, seed=g.Hq, utility0="exp")
        if kind == "value":
            for s, sign in ((0, 1.0), (1, -1.0)):
                case.V_shards[s][s, g.S - 1, 3] = sign * np.inf
        elif g.rank:                     # q and the decoder row of one code column positive: -Inf for all heads
            case.q, case.U_K[:, 7] = np.abs(case.q), np.abs(case.U_K[:, 7])
            case.K_shards[1][:, g.S - 1, 7] = -np.inf
        else:
            case.q[..., 5] = np.abs(case.q[..., 5])
            case.K_shards[1][:, g.S - 1, 5] = -np.inf
        ref = oracle_step(case, idx, gates, orc.COMBINE_LSE)["y"]
        assert np.isinf(ref).any() == (kind == "value") and not np.isnan(ref).any()
        dc = DeviceCase(case)
        dc.attend(topk=torch.from_numpy(idx).to(DEV), gates=torch.from_numpy(gates).to(DEV))
        y = t2n(dc.y)
        for what in (np.isposinf, np.isneginf, np.isnan):
            np.testing.assert_array_equal(what(y), what(ref), err_msg=kind)
        ok = np.isfinite(ref)
        assert np.linalg.norm(y[ok] - ref[ok]) <= 1e-6 * np.linalg.norm(ref[ok])


@pytest.mark.parametrize("spec", [
    dict(B=1, Hq=8, Hkv=2, D=128, E=12, S=2304, k=12, dtype="bf16"),       # matrix cores, 128 rows a round
    dict(B=1, Hq=6, Hkv=2, D=64, E=12, S=2051, k=12, dtype="bf16", rank=32),
    dict(B=1, Hq=2, Hkv=2, D=128, E=12, S=2304, k=12, dtype="bf16"),       # plain ALU
    dict(B=1, Hq=4, Hkv=2, D=64, E=12, S=1030, k=12, dtype="f32"),
    # a wave's last tile has a pass of its own (one, two and four heads) or none (eight)
    dict(B=1, Hq=2, Hkv=2, D=128, E=12, S=1030, k=12, dtype="f32"), dict(B=1, Hq=8, Hkv=2, D=64, E=12, S=1031, k=12, dtype="f32"),
    dict(B=1, Hq=8, Hkv=1, D=32, E=12, S=1030, k=12, dtype="f32"), dict(B=1, Hq=3, Hkv=1, D=128, E=12, S=1030, k=12, dtype="f32", rank=16),
    dict(B=1, Hq=2, Hkv=2, D=64, E=12, S=2051, k=12, dtype="bf16", rank=32),
], ids=lambda s: "G%d_%s_r%d" % (s["Hq"] // s["Hkv"], s["dtype"], s.get("rank", 0)))
@pytest.mark.parametrize("forced", [0, 5, 64])
def test_splits_follow_the_entry_count(spec, forced):
    """Shards that hold from nothing to their capacity, at the edges of a round of tiles and of a split:
    every split takes its share of the entries that are there, and the merge sees each of them once."""
    g = wl.Geometry(**spec)
    nv = np.array([[0, 1, 63, 64, 127, 128, 129, 255, 257, g.S // 2 + 1, g.S - 1, g.S]], np.int32)
    case = wl.make_host_case(g, seed=3, n_valid=nv, utility0="exp")
    idx, gates = random_selection(g, 4)
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE, utility=u_ref, decay=0.5)
    pk.pikv_set_attn_split(forced)
    try:
        dc = DeviceCase(case)
        d_idx, d_gates = torch.from_numpy(idx).to(DEV), torch.from_numpy(gates).to(DEV)
        dc.attend(topk=d_idx, gates=d_gates)
        dc.update_utility(0.5, topk=d_idx)
        y = t2n(dc.y)
    finally:
        pk.pikv_set_attn_split(0)
    assert np.linalg.norm(y - ref["y"]) <= 8e-6 * np.linalg.norm(ref["y"])
    assert_utility_close(t2n(dc.utility), u_ref)
    sc = t2n(dc.scores)
    for j in range(g.k):         # a score row is written up to the shard's count and not past it
        n = nv[0, idx[0, j]]
        assert np.isfinite(sc[0, :, j, :n]).all() and np.isnan(sc[0, :, j, n:]).all()


@pytest.mark.parametrize("spec", [
    # nearly the units for a block per CU, but many partials or long blocks: 60, 192 and 204 units
    dict(Hq=20, Hkv=5, D=128, S=4111, k=12), dict(Hq=32, Hkv=16, D=64, S=2304, k=12), dict(Hq=51, Hkv=17, D=64, S=2050, k=12),
    dict(Hq=48, Hkv=16, D=64, S=4500, k=12, rank=32), dict(Hq=64, Hkv=16, D=16, S=8200, k=12),
    # a block per CU: 108 units with two splits, 204 and 252 with one
    dict(Hq=36, Hkv=9, D=128, S=2003, k=12), dict(Hq=72, Hkv=9, D=128, S=2048, k=12), dict(Hq=18, Hkv=9, D=64, S=4091, k=12),
    dict(Hq=51, Hkv=17, D=64, S=2045, k=12), dict(Hq=63, Hkv=21, D=64, S=4001, k=12, rank=32), dict(Hq=84, Hkv=21, D=16, S=2040, k=12),
    # few units: a tile per wave, and blocks of fewer waves with rows than waves
    dict(Hq=8, Hkv=1, D=128, S=1030, k=2), dict(Hq=8, Hkv=1, D=64, S=938, k=7), dict(Hq=3, Hkv=3, D=128, S=600, k=3),
    dict(Hq=4, Hkv=1, D=128, S=258, k=1, rank=16), dict(Hq=20, Hkv=1, D=128, S=1000, k=1),
    dict(Hq=2, Hkv=2, D=64, S=700, k=2, dtype="f32"), dict(Hq=8, Hkv=1, D=128, S=300, k=1, dtype="f32"),
    dict(Hq=6, Hkv=2, D=64, S=515, k=2, rank=32, dtype="f32"),
], ids=lambda s: "%s_G%d_u%d_D%d_r%d_S%d" % (s.get("dtype", "bf16"), s["Hq"] // s["Hkv"], s["Hkv"] * s["k"], s["D"], s.get("rank", 0), s["S"]))
def test_few_and_whole_blocks_follow_the_entry_count(spec):
    """The same for the plans of few units (down to a tile per block) and of one block per CU."""
    test_splits_follow_the_entry_count(dict(dict(B=1, E=12, dtype="bf16"), **spec), 0)


@pytest.mark.parametrize("spec,tq", [
    (dict(Hq=2, D=128, S=40), 2), (dict(Hq=16, D=128, S=300), 2), (dict(Hq=64, D=128, S=9), 4), (dict(Hq=3, D=128, S=33), 1),
    (dict(Hq=2, D=16, S=40), 1), (dict(Hq=24, D=32, S=130), 1), (dict(Hq=4, D=64, S=700), 1),
    (dict(Hq=8, D=128, rank=16, S=40), 1), (dict(Hq=5, D=64, rank=64, S=77), 1),
], ids=lambda v: "tq%d" % v if isinstance(v, int) else "G%d_D%d_r%d_S%d" % (v["Hq"], v["D"], v.get("rank", 0), v["S"]))
@pytest.mark.parametrize("limit", ["below", "at"])
def test_rows_spread_over_4_GiB(spec, tq, limit):
    """A kv head whose rows span nearly 4 GiB (32-bit offsets in the matrix-core kernel, its requests past the
    end included) and one whose rows span it exactly (the plain kernel, groups of 2, 4 and 8 heads
    among them) give the bits of densely stored ones, or those of the same kernel's dense form."""
    g = wl.Geometry(B=1, Hkv=1, E=2, k=2, dtype="bf16", **spec)
    half = (1 << 31) // g.S // 8 * 8
    stride = half - 8 if limit == "below" else -(-(1 << 31) // g.S // 8) * 8
    if limit == "at" and tq > 1:       # no kernel takes draft queries there
        assert pk.pikv_attn_workspace_bytes(pk.make_desc(1, g.Hq, 1, g.D, 2, g.S, dtype=1, stride_s=stride, tq=tq), g.k) == 0
        return
    nv = np.array([[g.S, max(1, g.S - 3)]], np.int32)
    case = wl.make_host_case(g, seed=g.S, n_valid=nv, utility0="exp")
    idx, gates = random_selection(g, 1)
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE)
    d = DeviceCase(case)
    d_idx, d_gates = torch.from_numpy(idx).to(DEV), torch.from_numpy(gates).to(DEV)
    heap = torch.empty((g.S - 1) * stride + 4 * 1024, device=DEV, dtype=torch.bfloat16)   # all four shards, in each other's gaps
    # gaps hold what a wrong offset would be punished for
    heap.fill_(float("nan"))
    w = g.width
    shards = [heap[1024 * i:][:(g.S - 1) * stride + w].as_strided((g.S, w), (stride, 1)) for i in range(4)]
    for e in range(2):
        shards[e].copy_(d.K[e, 0, :g.S, :w])
        shards[2 + e].copy_(d.V[e, 0, :g.S, :w])
    d.K_tab, d.V_tab = pk.shard_table(shards[:2]), pk.shard_table(shards[2:])
    d.desc = pk.make_desc(1, g.Hq, 1, g.D, 2, g.S, rank=g.rank, dtype=pk.binding.BF16, stride_s=stride, stride_h=0, tq=tq)
    d.workspace = torch.empty(pk.pikv_attn_workspace_bytes(d.desc, g.k), device=DEV, dtype=torch.uint8)
    d.attend(topk=d_idx, gates=d_gates)
    y = t2n(d.y)
    assert np.linalg.norm(y - ref["y"]) <= (8e-6 if w == 128 else 1e-6) * np.linalg.norm(ref["y"])
    sc = t2n(d.scores)
    for j in range(2):
        n = nv[0, idx[0, j]]
        assert np.isfinite(sc[0, :, j, :n]).all() and np.isnan(sc[0, :, j, n:]).all()


def test_attention_is_bitwise_repeatable():
    spec, nv = ATTN_CASES["c3_scaled"]
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=12, n_valid=nv)
    idx, gates = random_selection(g, 6)
    dc = DeviceCase(case)
    d_idx, d_gates = torch.from_numpy(idx).to(DEV), torch.from_numpy(gates).to(DEV)
    outs = []
    for _ in range(2):
        dc.utility.zero_()
        dc.attend(topk=d_idx, gates=d_gates)
        dc.update_utility(1.0, topk=d_idx)
        outs.append((t2n(dc.y), t2n(dc.utility)))
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    np.testing.assert_array_equal(outs[0][1], outs[1][1])


def test_strided_shards_and_explicit_scale():
    g = wl.Geometry(B=1, Hq=4, Hkv=2, D=64, E=3, S=200, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=13, n_valid="ragged")
    idx, gates = random_selection(g, 7)
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE, scale=0.2)
    dc = DeviceCase(case, stride_pad=(8, 5))
    dc.attend(topk=torch.from_numpy(idx).to(DEV), gates=torch.from_numpy(gates).to(DEV), scale=0.2,
              want_scores=False)
    ok, emax, l2 = y_tolerance_ok(t2n(dc.y), ref["y"], g.dtype)
    assert ok, (emax, l2)


def test_all_selected_shards_empty_gives_zero_and_leaves_utility():
    g = wl.Geometry(B=2, Hq=4, Hkv=4, D=64, E=4, S=64, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=14, utility0="exp")
    case.n_valid[0, :] = 0
    case.n_valid[1, 2] = 0
    idx = np.array([[0, 1], [2, 3]], np.int32)
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, None, orc.COMBINE_LSE, utility=u_ref, decay=0.5)
    dc = DeviceCase(case)
    d_idx = torch.from_numpy(idx).to(DEV)
    dc.attend(topk=d_idx, gates=None)
    dc.update_utility(0.5, topk=d_idx)
    y = t2n(dc.y)
    assert (y[0] == 0).all()
    ok, emax, l2 = y_tolerance_ok(y, ref["y"], g.dtype)
    assert ok, (emax, l2)
    assert_utility_close(t2n(dc.utility), u_ref)
    np.testing.assert_array_equal(t2n(dc.utility)[0], case.utility[0])


# ---------------------------------------------------------------- evict / append
def run_gpu_evict(g, u, n, capacity, sel=None, max_evict=None, compact=False, case=None):
    dt = g.dtype
    if case is None:
        case = wl.make_host_case(g, seed=1)
    case = case.clone()
    case.utility, case.n_valid = u.copy(), n.copy()
    dc = DeviceCase(case)
    if max_evict is None:
        max_evict = max(1, g.S - capacity)
    eidx = torch.full((g.B, g.E, max_evict), -1, device=DEV, dtype=torch.int32)
    ecnt = torch.full((g.B, g.E), -7, device=DEV, dtype=torch.int32)
    d_sel = None if sel is None else torch.from_numpy(sel).to(DEV)
    pk.pikv_evict(dc.desc, dc.utility, dc.n_valid, capacity, d_sel, 0 if sel is None else sel.shape[1],
                  eidx, ecnt, max_evict, compact, dc.K_tab if compact else None,
                  dc.V_tab if compact else None)
    return dc, t2n(eidx), t2n(ecnt)


@pytest.mark.parametrize("S,capacity", [(256, 192), (1000, 1), (16, 6), (2048, 2047), (5000, 4096), (300, 0),
                                        (3000, 2000), (12000, 9000), (20000, 100), (40000, 30000), (1001, 700), (255, 100)])
@pytest.mark.parametrize("ties", [False, True], ids=["distinct", "ties"])
def test_evict_matches_oracle_bit_exact(S, capacity, ties):
    g = wl.Geometry(B=2, Hq=2, Hkv=2, D=16, E=3, S=S, k=2, dtype="bf16")
    rng = np.random.default_rng(S + capacity)
    if ties:
        u = (rng.integers(0, 6, size=(g.B, g.E, S)) / 8).astype(np.float32)
    else:
        u = (rng.exponential(1.0, size=(g.B, g.E, S)) / S).astype(np.float32)
    n = rng.integers(max(0, capacity - 3), S + 1, size=(g.B, g.E)).astype(np.int32)
    n[0, 0] = S
    u_ref, n_ref = u.copy(), n.copy()
    ridx, rcnt = orc.evict(u_ref, n_ref, capacity, max_evict=max(1, S - capacity))
    dc, eidx, ecnt = run_gpu_evict(g, u, n, capacity)
    np.testing.assert_array_equal(ecnt, rcnt)
    for b in range(g.B):
        for e in range(g.E):
            np.testing.assert_array_equal(eidx[b, e, :rcnt[b, e]], ridx[b, e, :rcnt[b, e]])
    np.testing.assert_array_equal(t2n(dc.n_valid), n_ref)
    np.testing.assert_array_equal(t2n(dc.utility), u_ref)


@pytest.mark.parametrize("S", [2047, 2048, 2049, 4099, 8192, 8193, 32768, 32771])
@pytest.mark.parametrize("ties", [False, True], ids=["distinct", "ties"])
def test_evict_matches_oracle_at_the_edges_of_the_select_shapes(S, ties):
    """Block sizes, keys per thread and rows that are not 16-byte aligned change at these capacities."""
    test_evict_matches_oracle_bit_exact(S, S * 3 // 4, ties)


@pytest.mark.parametrize("n", [2, 255, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("S", [2049, 2052, 9000])
@pytest.mark.parametrize("compact", [False, True], ids=["list", "compact"])
def test_evict_few_entries_of_a_large_shard(n, S, compact):
    """Up to 2048 entries take a quarter of the block, whatever the capacity; shards of both kinds in a call."""
    g = wl.Geometry(B=1, Hq=2, Hkv=2, D=16, E=4, S=S, k=2, dtype="bf16")
    rng = np.random.default_rng(n)
    u = (rng.integers(0, 900, size=(1, 4, S)) / 8 + 1).astype(np.float32)
    counts = np.array([[n, S, n // 2, max(1, n - 1)]], np.int32)
    capacity = max(1, n // 2)
    u_ref, n_ref = u.copy(), counts.copy()
    ridx, rcnt = orc.evict(u_ref, n_ref, capacity, max_evict=S)
    dc, eidx, ecnt = run_gpu_evict(g, u, counts, capacity, max_evict=S, compact=compact)
    np.testing.assert_array_equal(ecnt, rcnt)
    np.testing.assert_array_equal(t2n(dc.n_valid), n_ref)
    got_u = t2n(dc.utility)
    for e in range(4):
        np.testing.assert_array_equal(eidx[0, e, :rcnt[0, e]], ridx[0, e, :rcnt[0, e]])
        kept = np.delete(u[0, e, :counts[0, e]], ridx[0, e, :rcnt[0, e]]) if compact else u[0, e]
        np.testing.assert_array_equal(got_u[0, e, :kept.size], kept)


@pytest.mark.parametrize("n", [3, 1023, 2048, 2049, 8193, 33000])
@pytest.mark.parametrize("kind", ["clusters", "neighbours", "least", "extremes", "crowd"])
def test_evict_cut_at_every_depth_of_the_histogram(n, kind):
    """Utilities that end the select in its first, second, third or last round: two far clusters of neighbouring
    bit patterns, consecutive bit patterns, ties at the least value, infinities of both signs, one value
    that fills most of a bin - in registers and re-read from memory, against a stable sort."""
    rng = np.random.default_rng(n)
    if kind == "clusters":
        bits = np.where(rng.random(n) < 0.5, 0x00000100, 0x7f000000) + rng.integers(0, 64, n)
        u = bits.astype(np.uint32).view(np.float32)
    elif kind == "neighbours":
        u = (0x3f000000 + rng.permutation(n)).astype(np.uint32).view(np.float32)
    elif kind == "least":
        u = np.where(rng.random(n) < 0.6, 0.0, rng.exponential(1.0, n)).astype(np.float32)
    elif kind == "extremes":
        u = rng.normal(size=n).astype(np.float32)
        u[rng.random(n) < 0.2], u[rng.random(n) < 0.2] = np.inf, -np.inf
    else:
        u = np.where(rng.random(n) < 0.8, 0.25, rng.random(n)).astype(np.float32)
        u[0] = -1.0
    E, S = 3, n + 5
    desc = pk.make_desc(1, 1, 1, 16, E, S, dtype=1)
    order = np.lexsort((np.arange(n), -u))                       # utility descending, then slot ascending
    for drop in sorted({1, n // 5 + 1, n // 2, n - 1, n} - {0}):
        util = torch.zeros((1, E, S), device=DEV)
        util[0, 1, :n] = torch.from_numpy(u.copy()).to(DEV)
        nv = torch.tensor([[0, n, 0]], device=DEV, dtype=torch.int32)
        eidx = torch.full((1, E, n), -7, device=DEV, dtype=torch.int32)
        ecnt = torch.zeros((1, E), device=DEV, dtype=torch.int32)
        pk.pikv_evict(desc, util, nv, n - drop, None, 0, eidx, ecnt, n, False, None, None)
        assert t2n(ecnt).tolist() == [[0, drop, 0]] and t2n(nv).tolist() == [[0, n - drop, 0]]
        np.testing.assert_array_equal(t2n(eidx)[0, 1, :drop], np.sort(order[n - drop:]))


def test_evict_special_values_and_selection_list():
    g = wl.Geometry(B=2, Hq=2, Hkv=2, D=16, E=4, S=64, k=2, dtype="bf16")
    rng = np.random.default_rng(3)
    u = rng.standard_normal((g.B, g.E, g.S)).astype(np.float32)       # negative utilities too
    u[0, 1, ::3] = 0.0
    u[0, 1, 1::6] = -0.0
    u[1, 2, :] = 0.25                                                  # all equal
    n = np.full((g.B, g.E), g.S, np.int32)
    sel = np.array([[1, 3], [2, 0]], np.int32)
    mask = np.zeros((g.B, g.E), np.int32)
    for b in range(g.B):
        mask[b, sel[b]] = 1
    u_ref, n_ref = u.copy(), n.copy()
    ridx, rcnt = orc.evict(u_ref, n_ref, 40, shard_mask=mask, max_evict=24)
    dc, eidx, ecnt = run_gpu_evict(g, u, n, 40, sel=sel, max_evict=24)
    np.testing.assert_array_equal(ecnt, rcnt)
    np.testing.assert_array_equal(eidx[mask == 1], ridx[mask == 1])
    np.testing.assert_array_equal(t2n(dc.n_valid), n_ref)
    # more to evict than max_evict: shard untouched, count -1
    dc, eidx, ecnt = run_gpu_evict(g, u, n, 10, max_evict=5)
    assert (ecnt == -1).all() and (t2n(dc.n_valid) == g.S).all()


@pytest.mark.parametrize("spec", [
    dict(B=1, Hq=4, Hkv=4, D=64, E=4, S=256, k=2, dtype="f32", per_head_routing=True),   # config 1: 256 -> 192
    dict(B=2, Hq=4, Hkv=2, D=128, E=3, S=700, k=2, dtype="bf16"),
    dict(B=1, Hq=2, Hkv=2, D=128, E=2, S=300, k=2, dtype="bf16", rank=32),
    dict(B=1, Hq=2, Hkv=2, D=128, E=2, S=3000, k=2, dtype="bf16"),       # many passes of the row mover
    dict(B=1, Hq=2, Hkv=1, D=128, E=2, S=600, k=1, dtype="f32"),         # 512-byte rows
    dict(B=1, Hq=2, Hkv=2, D=16, E=2, S=2500, k=1, dtype="bf16"),        # 32-byte rows
], ids=["c1", "bf16_d128", "rank32", "bf16_s3000", "f32_d128", "bf16_d16"])
def test_evict_with_compaction_moves_rows_like_oracle(spec):
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=21, n_valid="ragged", utility0="exp")
    case.n_valid[0, 0] = g.S
    capacity = (g.S * 3) // 4
    ref = case.clone()
    ridx, rcnt = orc.evict(ref.utility, ref.n_valid, capacity, compact=True, K_shards=ref.K_shards,
                           V_shards=ref.V_shards, Hkv=g.Hkv, width=g.width, dtype=g.dtype)
    dc, eidx, ecnt = run_gpu_evict(g, case.utility, case.n_valid, capacity, compact=True, case=case)
    np.testing.assert_array_equal(ecnt, rcnt)
    n_new = t2n(dc.n_valid)
    np.testing.assert_array_equal(n_new, ref.n_valid)
    u = t2n(dc.utility)
    for b in range(g.B):
        for e in range(g.E):
            s, nn = b * g.E + e, n_new[b, e]
            np.testing.assert_array_equal(eidx[b, e, :rcnt[b, e]], ridx[b, e, :rcnt[b, e]])
            np.testing.assert_array_equal(u[b, e, :nn], ref.utility[b, e, :nn])
            np.testing.assert_array_equal(dc.shard_host("K", s)[:, :nn], ref.K_shards[s][:, :nn])
            np.testing.assert_array_equal(dc.shard_host("V", s)[:, :nn], ref.V_shards[s][:, :nn])


@pytest.mark.parametrize("S,cap,D,dtype,Hkv,E", [
    (513, 512, 16, "bf16", 1, 2),           # one row leaves; 256 threads
    (2048, 1536, 128, "bf16", 2, 3), (2561, 2048, 128, "f32", 1, 2), (4096, 1, 64, "bf16", 1, 2),
    (3000, 0, 64, "bf16", 2, 2),            # nothing is kept
    (30000, 10000, 32, "bf16", 1, 2),       # more evicted slots than the mover holds in LDS
    (40000, 30001, 128, "bf16", 7, 2),      # more than the Infinity Cache holds ...
    (40000, 30001, 128, "bf16", 7, 4),      # ... and past 512 MiB: the streaming form
    (1100, 300, 16, "bf16", 64, 16),        # 2048 blocks of a single pass: 256 threads
    (2100, 2099, 16, "bf16", 64, 16),       # as many of more than one pass
    (3000, 500, 128, "bf16", 2, 2),         # 64-byte column slices
], ids=lambda v: str(v))
@pytest.mark.parametrize("where", ["mixed", "tail", "head"])
def test_compaction_slides_rows_at_the_movers_edges(S, cap, D, dtype, Hkv, E, where):
    """Kept rows of K and V against an indexed copy, bit for bit, and nothing above the kept prefix changes:
    evicted slots everywhere, only at the end (nothing moves) and only at the start (all rows move)."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(S + D)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.empty((1, E, Hkv, S, D), device=DEV, dtype=tdt).normal_(generator=gen)
    V = torch.empty_like(K).normal_(generator=gen)
    n = torch.tensor([[S] + [max(1, S - 77)] * (E - 1)], device=DEV, dtype=torch.int32)
    u = torch.rand((1, E, S), device=DEV, generator=gen) + 0.5
    if where == "tail":
        u[:] = torch.arange(S, 0, -1, device=DEV)
    elif where == "head":
        u[:] = torch.arange(1, S + 1, device=DEV)
    wantK, wantV, gone = K.clone(), V.clone(), {}
    for e in range(E):
        ne = int(n[0, e])
        if ne > cap:
            order = torch.argsort(u[0, e, :ne], descending=True, stable=True)
            keep, gone[e] = order[:cap].sort().values, order[cap:].sort().values
            wantK[0, e, :, :cap], wantV[0, e, :, :cap] = K[0, e][:, keep], V[0, e][:, keep]
    drop = S - cap
    eidx = torch.full((1, E, drop), -1, device=DEV, dtype=torch.int32)
    ecnt = torch.zeros((1, E), device=DEV, dtype=torch.int32)
    desc = pk.make_desc(1, Hkv, Hkv, D, E, S, dtype=pk.binding.F32 if dtype == "f32" else pk.binding.BF16)
    pk.pikv_evict(desc, u, n, cap, None, 0, eidx, ecnt, drop, True, pk.shard_table(K), pk.shard_table(V))
    assert torch.equal(K, wantK) and torch.equal(V, wantV)
    for e, slots in gone.items():
        assert int(ecnt[0, e]) == slots.numel() and torch.equal(eidx[0, e, :slots.numel()], slots.int())


def test_append_matches_oracle_bit_exact():
    g = wl.Geometry(B=3, Hq=4, Hkv=2, D=128, E=4, S=50, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=22, n_valid="ragged", utility0="exp")
    case.n_valid[1, 1] = g.S                                # a full shard: entry dropped
    idx = np.array([[0, 2], [1, 3], [3, 0]], np.int32)
    kn, vn = wl.draw_new_kv(g, 5)
    from gpu_harness import dev_storage
    dc = DeviceCase(case)
    pk.pikv_append(dc.desc, dev_storage(kn, g.dtype), dev_storage(vn, g.dtype),
                   torch.from_numpy(idx).to(DEV), g.k, None, None, 0, dc.K_tab, dc.V_tab,
                   dc.utility, dc.n_valid)
    ref = case.clone()
    # the oracle reports a full shard as an error; the library drops the entry for that shard
    idx_ok = idx.copy()
    ref_n_full = ref.n_valid.copy()
    for b in range(g.B):
        sel = [e for e in idx[b] if ref.n_valid[b, e] < g.S]
        for e in sel:
            one = np.array([[e]], np.int32)
            orc.append(np.ascontiguousarray(kn[b:b + 1]), np.ascontiguousarray(vn[b:b + 1]), one,
                       ref.K_shards[b * g.E:(b + 1) * g.E], ref.V_shards[b * g.E:(b + 1) * g.E],
                       ref.utility[b:b + 1], ref.n_valid[b:b + 1], dtype=g.dtype)
    np.testing.assert_array_equal(t2n(dc.n_valid), ref.n_valid)
    np.testing.assert_array_equal(t2n(dc.utility), ref.utility)
    for s in range(g.B * g.E):
        np.testing.assert_array_equal(dc.shard_host("K", s), ref.K_shards[s])
        np.testing.assert_array_equal(dc.shard_host("V", s), ref.V_shards[s])
    assert ref.n_valid[1, 1] == g.S and idx_ok is not None and ref_n_full is not None


# --------------------------------------------------------- streaming (config 4, scaled)
def test_streaming_steps_route_evict_append_attend_update():
    """Each step: route -> evict the min-utility entry of every selected full shard ->
    append the new token there -> attend -> utility with decay 0.9.  The GPU carries its own
    state; at every step its selections and evicted slots must equal the oracle's applied
    to the GPU's own pre-step bits, and the free-running oracle state must stay within
    tolerance."""
    g = wl.Geometry(B=4, Hq=4, Hkv=4, D=64, E=4, S=96, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=31, utility0="exp")
    case.n_valid[:, 0] = g.S - 2                      # some shards still have room
    from gpu_harness import dev_storage
    dc = DeviceCase(case)
    eidx = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
    ecnt = torch.zeros((g.B, g.E), device=DEV, dtype=torch.int32)
    ref = case.clone()
    for step in range(12):
        qn = wl.draw_queries(g, 500 + step)
        probe = case.clone()
        probe.q = qn
        ensure_route_margin(probe, g.k)
        qn = probe.q
        kn, vn = wl.draw_new_kv(g, 900 + step)
        # --- GPU
        dc.q.copy_(dev_storage(qn, g.dtype))
        u_before, n_before = t2n(dc.utility), t2n(dc.n_valid)
        dc.route()
        pk.pikv_evict(dc.desc, dc.utility, dc.n_valid, g.S - 1, dc.topk, g.k, eidx, ecnt, 1, False,
                      None, None)
        pk.pikv_append(dc.desc, dev_storage(kn, g.dtype), dev_storage(vn, g.dtype), dc.topk, g.k,
                       eidx, ecnt, 1, dc.K_tab, dc.V_tab, dc.utility, dc.n_valid)
        dc.attend(combine=pk.COMBINE_LSE)
        dc.update_utility(0.9)
        # --- oracle, free running
        x = np.ascontiguousarray(qn.reshape(g.route_rows, g.d_r))
        idx, gates, _ = orc.route(x, ref.W_r, g.k, dtype=g.dtype)
        np.testing.assert_array_equal(t2n(dc.topk), idx)
        mask = np.zeros((g.B, g.E), np.int32)
        for b in range(g.B):
            mask[b, idx[b]] = 1
        # evict parity on identical bits: the oracle applied to the GPU's own pre-step state
        ub, nb = u_before.copy(), n_before.copy()
        pidx, pcnt = orc.evict(ub, nb, g.S - 1, shard_mask=mask, max_evict=1)
        np.testing.assert_array_equal(t2n(ecnt), pcnt)
        np.testing.assert_array_equal(t2n(eidx)[pcnt == 1], pidx[pcnt == 1])
        ridx, rcnt = orc.evict(ref.utility, ref.n_valid, g.S - 1, shard_mask=mask, max_evict=1)
        np.testing.assert_array_equal(rcnt, pcnt)
        assert (ridx[rcnt == 1] == pidx[pcnt == 1]).all(), "free-running oracle diverged at step %d" % step
        orc.append(kn, vn, idx, ref.K_shards, ref.V_shards, ref.utility, ref.n_valid, dtype=g.dtype,
                   reuse_idx=ridx, reuse_cnt=rcnt)
        ref.q = qn
        out = oracle_step(ref, idx, gates, orc.COMBINE_LSE, utility=ref.utility, decay=0.9)
        ok, emax, l2 = y_tolerance_ok(t2n(dc.y), out["y"], g.dtype)
        assert ok, (step, emax, l2)
        assert_utility_close(t2n(dc.utility), ref.utility)
        np.testing.assert_array_equal(t2n(dc.n_valid), ref.n_valid)
        assert (ref.n_valid <= g.S).all()
    for s in range(g.B * g.E):
        np.testing.assert_array_equal(dc.shard_host("K", s), ref.K_shards[s])


# ------------------------------------------------------------------- fused decode step
@pytest.mark.parametrize("spec", [
    dict(B=4, Hq=4, Hkv=4, D=64, E=8, S=96, k=2, dtype="bf16"),
    dict(B=2, Hq=8, Hkv=2, D=128, E=16, S=200, k=4, dtype="bf16"),
    dict(B=3, Hq=4, Hkv=4, D=128, E=8, S=64, k=5, dtype="bf16", rank=32),
    dict(B=2, Hq=4, Hkv=2, D=64, E=4, S=50, k=2, dtype="f32"),
    dict(B=2, Hq=8, Hkv=2, D=128, E=12, S=120, k=3, dtype="bf16"),       # W_r rows of 24 bytes: generic router
    dict(B=1, Hq=4, Hkv=4, D=64, E=2, S=70, k=2, dtype="bf16"),          # ... of 4 bytes
    # many sequences: more blocks in the step's first kernel than the GPU has compute units
    dict(B=36, Hq=4, Hkv=4, D=64, E=8, S=40, k=2, dtype="bf16"),
    dict(B=90, Hq=2, Hkv=2, D=32, E=3, S=24, k=2, dtype="f32"),
], ids=["g1", "gqa4", "rank32_k5", "f32", "e12", "e2", "b36_e8", "b90_e3_f32"])
def test_fused_decode_step_equals_separate_calls_and_oracle(spec):
    """pikv_decode_step (3 launches) vs the five separate calls (bit-identical state) vs oracle."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=41, utility0="exp", zipf_s=1.1)
    case.n_valid[:, 0] = g.S - 3                       # a shard with room
    dA, dB = DeviceCase(case), DeviceCase(case)
    eiA = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
    ecA = torch.full((g.B, g.E), -5, device=DEV, dtype=torch.int32)
    eiB, ecB = eiA.clone(), ecA.clone()
    ref = case.clone()
    for step in range(6):
        probe = case.clone()
        probe.q = wl.draw_queries(g, 700 + step)
        ensure_route_margin(probe, g.k)
        qn = probe.q
        kn, vn = wl.draw_new_kv(g, 800 + step)
        dkn, dvn = dev_storage(kn, g.dtype), dev_storage(vn, g.dtype)
        for d in (dA, dB):
            d.q.copy_(dev_storage(qn, g.dtype))
        # A: fused
        pk.pikv_decode_step(dA.desc, dA.q, dA.W_r, dA.bias, dkn, dvn, dA.K_tab, dA.V_tab, dA.U_K, dA.U_V,
                            dA.n_valid, dA.utility, g.k, pk.COMBINE_LSE, 0.0, 0.9, dA.topk, dA.gates,
                            eiA, ecA, dA.y, dA.row_max, dA.row_norm, dA.scores, dA.slot_coef, dA.workspace)
        # B: separate calls
        dB.route()
        pk.pikv_evict(dB.desc, dB.utility, dB.n_valid, g.S - 1, dB.topk, g.k, eiB, ecB, 1, False, None, None)
        pk.pikv_append(dB.desc, dkn, dvn, dB.topk, g.k, eiB, ecB, 1, dB.K_tab, dB.V_tab, dB.utility, dB.n_valid)
        dB.attend(combine=pk.COMBINE_LSE)
        dB.update_utility(0.9)
        for name in ("topk", "gates", "n_valid", "utility", "y", "K", "V"):
            a, b2 = getattr(dA, name), getattr(dB, name)
            if a.dtype == torch.bfloat16:
                a, b2 = a.view(torch.int16), b2.view(torch.int16)
            np.testing.assert_array_equal(t2n(a), t2n(b2), err_msg="%s differs at step %d" % (name, step))
        np.testing.assert_array_equal(t2n(ecA), t2n(ecB))
        np.testing.assert_array_equal(t2n(eiA)[t2n(ecA) == 1], t2n(eiB)[t2n(ecB) == 1])
        # oracle, free running
        x = np.ascontiguousarray(qn.reshape(g.route_rows, g.d_r))
        idx, gates, _ = orc.route(x, ref.W_r, g.k, bias=ref.bias, dtype=g.dtype)
        np.testing.assert_array_equal(t2n(dA.topk), idx)
        mask = np.zeros((g.B, g.E), np.int32)
        for b in range(g.B):
            mask[b, idx[b]] = 1
        ridx, rcnt = orc.evict(ref.utility, ref.n_valid, g.S - 1, shard_mask=mask, max_evict=1)
        np.testing.assert_array_equal(t2n(ecA), rcnt)
        orc.append(kn, vn, idx, ref.K_shards, ref.V_shards, ref.utility, ref.n_valid, dtype=g.dtype,
                   reuse_idx=ridx, reuse_cnt=rcnt)
        ref.q = qn
        out = oracle_step(ref, idx, gates, orc.COMBINE_LSE, utility=ref.utility, decay=0.9)
        ok, emax, l2 = y_tolerance_ok(t2n(dA.y), out["y"], g.dtype)
        assert ok, (step, emax, l2)
        assert_utility_close(t2n(dA.utility), ref.utility)
        np.testing.assert_array_equal(t2n(dA.n_valid), ref.n_valid)


@pytest.mark.parametrize("bad", ["workspace_alignment", "workspace_size", "nan_scale", "missing_decoder"])
def test_rejected_fused_step_leaves_the_cache_untouched(bad):
    """Argument errors of the attention pass are found before the step's first launch: after a
    rejected call no row, utility, entry count or routing output has changed."""
    from gpu_harness import dev_storage
    spec = dict(B=2, Hq=4, Hkv=4, D=128, E=8, S=64, k=2, dtype="bf16")
    if bad == "missing_decoder":
        spec["rank"] = 32
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=5, utility0="exp")
    d = DeviceCase(case)
    kn, vn = wl.draw_new_kv(g, 6)
    dkn, dvn = dev_storage(kn, g.dtype), dev_storage(vn, g.dtype)
    ei = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
    ec = torch.full((g.B, g.E), -5, device=DEV, dtype=torch.int32)
    d.topk.fill_(-7)
    ws, scale, U_K, U_V = d.workspace, 0.0, d.U_K, d.U_V
    if bad == "workspace_alignment":
        big = torch.empty(d.workspace.numel() + 256, device=DEV, dtype=torch.uint8)
        ws = big[16:16 + d.workspace.numel()]
    elif bad == "workspace_size":
        ws = d.workspace[:d.workspace.numel() // 2]
    elif bad == "nan_scale":
        scale = float("nan")
    else:
        U_K = U_V = None
    before = {n: t2n(getattr(d, n).view(torch.int16) if getattr(d, n).dtype == torch.bfloat16 else getattr(d, n))
              for n in ("K", "V", "utility", "n_valid", "topk")}
    with pytest.raises(pk.PikvError) as err:
        pk.pikv_decode_step(d.desc, d.q, d.W_r, d.bias, dkn, dvn, d.K_tab, d.V_tab, U_K, U_V, d.n_valid,
                            d.utility, g.k, pk.COMBINE_LSE, scale, 1.0, d.topk, d.gates, ei, ec, d.y,
                            d.row_max, d.row_norm, d.scores, d.slot_coef, ws)
    assert err.value.status == (-3 if bad == "workspace_size" else -1)
    torch.cuda.synchronize()
    for n, ref in before.items():
        t = getattr(d, n)
        np.testing.assert_array_equal(t2n(t.view(torch.int16) if t.dtype == torch.bfloat16 else t), ref, err_msg=n)
    assert (t2n(ec) == -5).all() and (t2n(ei) == -1).all()


@pytest.mark.gpu
@pytest.mark.parametrize("S", [8, 260, 4096 + 8, 2 * 8192 + 4], ids=lambda S: "S%d" % S)
def test_fused_step_evicts_the_oracles_victim_on_ties_zeros_and_negative_utilities(S):
    """The fused step's scan against the eviction rule on values chosen to separate its cases: every
    shard full; per shard all utilities equal, zeros of both signs, duplicated minima at the ends of
    the threads' ranges, negative values and infinities, ordinary positive ones (S: less than one
    load per thread, a partial pass, one pass and a bit, two passes and a bit)."""
    from gpu_harness import dev_storage
    g = wl.Geometry(B=2, Hq=2, Hkv=2, D=32, E=8, S=S, k=8, dtype="bf16")      # every shard is visited
    case = wl.make_host_case(g, seed=77, utility0="exp")
    rng = np.random.default_rng(S)
    u = np.abs(rng.standard_normal((g.B, g.E, S))).astype(np.float32) + 0.5
    u[0, 0, :] = 0.25                                  # all equal: the highest slot goes
    u[0, 1, ::3] = 0.0
    u[0, 1, 1::6] = -0.0                               # a sign bit, and equal to +0 in the order
    lo = np.float32(0.125)
    u[0, 2, [0, S // 2, S - 1]] = lo                   # the minimum three times
    u[0, 3, :] = rng.standard_normal(S).astype(np.float32)         # negative values
    u[0, 4, S // 3] = -np.inf
    u[0, 5, :] = np.inf
    u[0, 5, S // 2] = 3.0e38
    u[0, 6, [3, 4 % S]] = np.float32(1e-45)            # denormals, adjacent slots of two loads
    u[1, 0, S - 1] = lo
    u[1, 1, 0] = lo
    u[1, 2, :] = 0.0                                   # all zero, as after a run of inserts
    u[1, 3, S - 4:] = lo                               # the last load, all four
    case.utility[:] = u
    case.n_valid[:] = S
    dc = DeviceCase(case)
    ei = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
    ec = torch.full((g.B, g.E), -5, device=DEV, dtype=torch.int32)
    kn, vn = wl.draw_new_kv(g, 5)
    pk.pikv_decode_step(dc.desc, dc.q, dc.W_r, dc.bias, dev_storage(kn, g.dtype), dev_storage(vn, g.dtype),
                        dc.K_tab, dc.V_tab, dc.U_K, dc.U_V, dc.n_valid, dc.utility, g.k, pk.COMBINE_LSE, 0.0, 1.0,
                        dc.topk, dc.gates, ei, ec, dc.y, dc.row_max, dc.row_norm, dc.scores, dc.slot_coef,
                        dc.workspace)
    ridx, rcnt = orc.evict(u.copy(), np.full((g.B, g.E), S, np.int32), S - 1, max_evict=1)
    assert (rcnt == 1).all()
    np.testing.assert_array_equal(t2n(ec), rcnt)
    np.testing.assert_array_equal(t2n(ei), ridx)
    assert ridx[0, 0, 0] == S - 1 and ridx[0, 2, 0] == S - 1 and ridx[1, 1, 0] == 0 and ridx[1, 2, 0] == S - 1


@pytest.mark.parametrize("seed", range(12))
def test_fused_step_is_bit_identical_to_separate_calls_on_random_geometries(seed):
    """The fused step is defined as the sequence of the separate calls: same bits in every piece of
    state after several steps, on shapes nobody hand-picked (both combine modes, decay, fills)."""
    from gpu_harness import dev_storage
    rng = np.random.default_rng(2000 + seed)
    dtype = str(rng.choice(["bf16", "bf16", "f32"]))
    # (expert counts whose W_r rows are whole aligned 16-byte chunks, and others: the router's
    # generic form inside the step)
    E = int(rng.choice([8, 16, 32, 5, 12, 24, 33] if dtype == "bf16" else [4, 8, 16, 3, 6, 13]))
    D = int(rng.choice([32, 64, 128]))
    rank = int(rng.choice([0, 0, 16, 32]))
    if rank >= D:
        rank = 0
    Hkv = int(rng.choice([1, 2, 4]))
    G = int(rng.choice([1, 2, 3, 4, 8]))
    g = wl.Geometry(B=int(rng.integers(1, 4)), Hq=Hkv * G, Hkv=Hkv, D=D, E=E, S=int(rng.integers(2, 300)),
                    k=int(rng.integers(1, min(E, 6) + 1)), dtype=dtype, rank=rank)
    case = wl.make_host_case(g, seed=seed, utility0="exp", zipf_s=1.1, n_valid=str(rng.choice(["ragged", "full"])))
    combine = int(rng.choice([pk.COMBINE_LSE, pk.COMBINE_LOCAL]))
    decay = float(rng.choice([1.0, 0.9, 0.5]))
    dA, dB = DeviceCase(case), DeviceCase(case)
    eiA = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
    ecA = torch.full((g.B, g.E), -5, device=DEV, dtype=torch.int32)
    eiB, ecB = eiA.clone(), ecA.clone()
    for step in range(4):
        qn = wl.draw_queries(g, 3000 + 10 * seed + step)
        kn, vn = wl.draw_new_kv(g, 4000 + 10 * seed + step)
        dkn, dvn = dev_storage(kn, g.dtype), dev_storage(vn, g.dtype)
        for d in (dA, dB):
            d.q.copy_(dev_storage(qn, g.dtype))
        pk.pikv_decode_step(dA.desc, dA.q, dA.W_r, dA.bias, dkn, dvn, dA.K_tab, dA.V_tab, dA.U_K, dA.U_V,
                            dA.n_valid, dA.utility, g.k, combine, 0.0, decay, dA.topk, dA.gates,
                            eiA, ecA, dA.y, dA.row_max, dA.row_norm, dA.scores, dA.slot_coef, dA.workspace)
        dB.route()
        pk.pikv_evict(dB.desc, dB.utility, dB.n_valid, g.S - 1, dB.topk, g.k, eiB, ecB, 1, False, None, None)
        pk.pikv_append(dB.desc, dkn, dvn, dB.topk, g.k, eiB, ecB, 1, dB.K_tab, dB.V_tab, dB.utility, dB.n_valid)
        dB.attend(combine=combine)
        dB.update_utility(decay)
        for name in ("topk", "gates", "n_valid", "utility", "y", "row_max", "row_norm", "K", "V"):
            a, b2 = getattr(dA, name), getattr(dB, name)
            if a.dtype == torch.bfloat16:
                a, b2 = a.view(torch.int16), b2.view(torch.int16)
            np.testing.assert_array_equal(t2n(a), t2n(b2), err_msg="%s differs at step %d for %s" % (name, step, g))
        np.testing.assert_array_equal(t2n(ecA), t2n(ecB))
        np.testing.assert_array_equal(t2n(eiA)[t2n(ecA) == 1], t2n(eiB)[t2n(ecB) == 1])


def test_fused_decode_step_without_insert_and_unsupported_shapes():
    g = wl.Geometry(B=2, Hq=4, Hkv=4, D=64, E=8, S=80, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=42, utility0="exp")
    ensure_route_margin(case, g.k)
    dA, dB = DeviceCase(case), DeviceCase(case)
    pk.pikv_decode_step(dA.desc, dA.q, dA.W_r, dA.bias, None, None, dA.K_tab, dA.V_tab, None, None,
                        dA.n_valid, dA.utility, g.k, pk.COMBINE_LOCAL, 0.0, 1.0, dA.topk, dA.gates,
                        None, None, dA.y, dA.row_max, dA.row_norm, dA.scores, dA.slot_coef, dA.workspace)
    dB.route()
    dB.attend(combine=pk.COMBINE_LOCAL)
    dB.update_utility(1.0)
    for name in ("topk", "y", "utility", "n_valid"):
        np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)))
    # per-head routing is not served by the fused step
    g2 = wl.Geometry(B=1, Hq=4, Hkv=4, D=64, E=4, S=32, k=2, dtype="f32", per_head_routing=True)
    d2 = DeviceCase(wl.make_host_case(g2, seed=1))
    with pytest.raises(pk.PikvError) as ei:
        pk.pikv_decode_step(d2.desc, d2.q, d2.W_r, None, None, None, d2.K_tab, d2.V_tab, None, None,
                            d2.n_valid, d2.utility, g2.k, pk.COMBINE_LSE, 0.0, 1.0, d2.topk, d2.gates,
                            None, None, d2.y, d2.row_max, d2.row_norm, d2.scores, d2.slot_coef, d2.workspace)
    assert ei.value.status == -2


# ------------------------------------------------ widened rows: router penalties, compress-on-insert
@pytest.mark.parametrize("mode", [0, 1, 2], ids=["load_balance", "cache_aware", "entropy"])
def test_router_penalty_matches_oracle_and_closes_the_loop(mode):
    """Table 1 penalty terms kept on the device: counters exact, bias to fp32 rounding, and the
    penalised routing decisions of a 10-step chain equal the oracle's."""
    from gpu_harness import dev_storage
    g = wl.Geometry(B=6, Hq=4, Hkv=4, D=64, E=8, S=16, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=51)
    dc = DeviceCase(case)
    rng = np.random.default_rng(3)
    miss_h = rng.integers(0, 50, size=g.E).astype(np.int32)
    load_h = np.zeros(g.E, np.int32)
    load_d = torch.zeros(g.E, device=DEV, dtype=torch.int32)
    miss_d = torch.from_numpy(miss_h).to(DEV)
    bias_d = torch.zeros(g.E, device=DEV)
    dc.bias = bias_d
    coef = (0.05, 0.3, 4.0)[mode]
    bias_h = np.zeros(g.E, np.float32)
    for step in range(10):
        probe = case.clone()
        probe.q = wl.draw_queries(g, 300 + step)
        probe.bias = bias_h
        ensure_route_margin(probe, g.k)
        dc.q.copy_(dev_storage(probe.q, g.dtype))
        dc.route()
        x = np.ascontiguousarray(probe.q.reshape(g.route_rows, g.d_r))
        idx, _, _ = orc.route(x, case.W_r, g.k, bias=bias_h, dtype=g.dtype)
        np.testing.assert_array_equal(t2n(dc.topk), idx)
        pk.pikv_router_penalty(mode, dc.topk, g.route_rows, g.k, g.E, load_d, miss_d, coef, bias_d)
        bias_h = orc.router_penalty(mode, idx, load_h, coef, miss=miss_h)
        np.testing.assert_array_equal(t2n(load_d), load_h)
        np.testing.assert_allclose(t2n(bias_d), bias_h, rtol=1e-5, atol=1e-6)
    assert load_h.sum() == 10 * g.route_rows * g.k


@pytest.mark.parametrize("mode", [0, 1, 2], ids=["load_balance", "cache_aware", "entropy"])
def test_router_feedback_inside_the_fused_step_equals_the_separate_penalty_call(mode):
    """pikv_decode_step_policy with a pikv_router_feedback: the step's last launch updates the
    load counters and the next step's bias exactly as pikv_router_penalty after the step would
    (same bits, every step of a closed loop), and the loop's selections equal the oracle's."""
    from gpu_harness import dev_storage
    g = wl.Geometry(B=5, Hq=8, Hkv=4, D=64, E=8, S=40, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=52, utility0="exp")
    dA, dB = DeviceCase(case), DeviceCase(case)
    rng = np.random.default_rng(4)
    miss_h = rng.integers(0, 50, size=g.E).astype(np.int32)
    coef = (0.05, 0.3, 4.0)[mode]
    state = {}
    for name, d in (("A", dA), ("B", dB)):
        state[name] = dict(load=torch.zeros(g.E, device=DEV, dtype=torch.int32), miss=torch.from_numpy(miss_h).to(DEV),
                           bias=torch.zeros(g.E, device=DEV),
                           ei=torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32),
                           ec=torch.zeros((g.B, g.E), device=DEV, dtype=torch.int32))
        d.bias = state[name]["bias"]
    fb = pk.make_router_feedback(mode, coef, state["A"]["load"], state["A"]["bias"], miss=state["A"]["miss"])
    load_h, bias_h = np.zeros(g.E, np.int32), np.zeros(g.E, np.float32)
    for step in range(8):
        probe = case.clone()
        probe.q = wl.draw_queries(g, 400 + step)
        probe.bias = bias_h
        ensure_route_margin(probe, g.k)
        kn, vn = wl.draw_new_kv(g, 450 + step)
        dkn, dvn = dev_storage(kn, g.dtype), dev_storage(vn, g.dtype)
        for d in (dA, dB):
            d.q.copy_(dev_storage(probe.q, g.dtype))
        sA, sB = state["A"], state["B"]
        pk.pikv_decode_step_policy(dA.desc, dA.q, dA.W_r, dA.bias, dkn, dvn, dA.K_tab, dA.V_tab, None, None,
                                   dA.n_valid, dA.utility, g.k, pk.COMBINE_LSE, 0.0, 0.9, dA.topk, dA.gates,
                                   sA["ei"], sA["ec"], dA.y, dA.row_max, dA.row_norm, dA.scores, dA.slot_coef,
                                   dA.workspace, None, feedback=fb)
        pk.pikv_decode_step(dB.desc, dB.q, dB.W_r, dB.bias, dkn, dvn, dB.K_tab, dB.V_tab, None, None,
                            dB.n_valid, dB.utility, g.k, pk.COMBINE_LSE, 0.0, 0.9, dB.topk, dB.gates,
                            sB["ei"], sB["ec"], dB.y, dB.row_max, dB.row_norm, dB.scores, dB.slot_coef,
                            dB.workspace)
        pk.pikv_router_penalty(mode, dB.topk, g.route_rows, g.k, g.E, sB["load"], sB["miss"], coef, sB["bias"])
        for name in ("topk", "y", "utility", "n_valid"):
            np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)), err_msg=name)
        np.testing.assert_array_equal(t2n(sA["load"]), t2n(sB["load"]))
        np.testing.assert_array_equal(t2n(sA["bias"]).view(np.uint32), t2n(sB["bias"]).view(np.uint32))
        # the oracle's closed loop
        x = np.ascontiguousarray(probe.q.reshape(g.route_rows, g.d_r))
        idx, _, _ = orc.route(x, case.W_r, g.k, bias=bias_h, dtype=g.dtype)
        np.testing.assert_array_equal(t2n(dA.topk), idx)
        bias_h = orc.router_penalty(mode, idx, load_h, coef, miss=miss_h)
        np.testing.assert_array_equal(t2n(sA["load"]), load_h)
        np.testing.assert_allclose(t2n(sA["bias"]), bias_h, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("spec", [
    dict(B=3, Hq=4, Hkv=4, D=128, E=4, S=300, k=2, dtype="bf16", rank=32),
    dict(B=2, Hq=8, Hkv=2, D=64, E=4, S=130, k=3, dtype="f32", rank=16),
    dict(B=2, Hq=4, Hkv=4, D=128, E=3, S=200, k=2, dtype="bf16", rank=64),
], ids=["bf16_r32", "f32_r16_gqa4", "bf16_r64"])
@pytest.mark.parametrize("combine", [orc.COMBINE_LSE, orc.COMBINE_LOCAL], ids=["lse", "local"])
def test_value_decoder_bias_matches_oracle(spec, combine):
    """Table 2 row LoRA++ on the value side: U_V carries one more row per kv head, the additive
    term of the decoder; outputs against the oracle's explicit decode with that term, an empty
    selection still gives zero, utilities are those of the run without the term."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=61, n_valid="ragged", utility0="exp")
    case.n_valid[-1, :] = 0                                   # the last sequence: every shard empty
    ensure_route_margin(case, g.k)
    rng = np.random.default_rng(62)
    b_V = wl.encode(rng.standard_normal((g.Hkv, g.D)), g.dtype)
    dc = DeviceCase(case)
    UVb = np.concatenate([case.U_V, b_V[:, None, :]], axis=1)            # [Hkv, rank + 1, D]
    dc.U_V = dev_storage(np.ascontiguousarray(UVb), g.dtype)
    dc.desc = pk.make_desc(g.B, g.Hq, g.Hkv, g.D, g.E, g.S, rank=g.rank,
                           dtype=pk.binding.F32 if g.dtype == "f32" else pk.binding.BF16,
                           stride_h=dc.stride_h, stride_s=dc.stride_s, flags=pk.DESC_VALUE_BIAS)
    dc.route()
    dc.attend(combine=combine)
    dc.update_utility(1.0)
    idx, gates = t2n(dc.topk), t2n(dc.gates)
    u_ref = case.utility.copy()
    ref = orc.attend(case.q, case.K_shards, case.V_shards, case.n_valid, idx, gates, Hkv=g.Hkv, E=g.E, S=g.S,
                     dtype=g.dtype, rank=g.rank, U_K=case.U_K, U_V=case.U_V, V_bias=b_V, combine=combine,
                     utility=u_ref)
    y = t2n(dc.y)
    ok, emax, l2 = y_tolerance_ok(y, ref["y"], g.dtype)
    assert ok, (emax, l2)
    assert (y[-1] == 0).all()
    assert_utility_close(t2n(dc.utility), u_ref)
    # and the difference to the run without the term is the term itself
    plain = DeviceCase(case)
    plain.route()
    plain.attend(combine=combine)
    diff = y[:-1] - t2n(plain.y)[:-1]
    want = wl.decode(b_V, g.dtype)[np.arange(g.Hq) // (g.Hq // g.Hkv)][None]
    np.testing.assert_allclose(diff, np.broadcast_to(want, diff.shape), rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("spec", [
    dict(B=16, Hq=32, Hkv=32, D=128, E=2, S=8, k=1, dtype="bf16", rank=32),     # config-5 shape
    dict(B=3, Hq=4, Hkv=2, D=64, E=2, S=8, k=1, dtype="bf16", rank=16),
    dict(B=2, Hq=2, Hkv=2, D=128, E=2, S=8, k=1, dtype="f32", rank=64),
], ids=["c5_shape", "rank16", "f32_rank64"])
def test_compress_matches_oracle(spec):
    """codes = W_enc x: fp32 storage to rounding error; bf16 storage equal to the oracle's
    round-to-nearest-even code except where fp32 vs fp64 summation straddles a rounding
    boundary (then exactly one bf16 step away)."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    rng = np.random.default_rng(9)
    x = wl.encode(rng.standard_normal((g.B, g.Hkv, g.D)), g.dtype)
    W = wl.encode(rng.standard_normal((g.Hkv, g.rank, g.D)) / np.sqrt(g.D), g.dtype)
    ref = orc.compress(x, W, dtype=g.dtype)
    desc = pk.make_desc(g.B, g.Hq, g.Hkv, g.D, g.E, g.S, rank=g.rank,
                        dtype=pk.binding.F32 if g.dtype == "f32" else pk.binding.BF16)
    out = torch.zeros((g.B, g.Hkv, g.rank), device=DEV,
                      dtype=torch.float32 if g.dtype == "f32" else torch.bfloat16)
    pk.pikv_compress(desc, dev_storage(x, g.dtype), dev_storage(W, g.dtype), out)
    torch.cuda.synchronize()
    got = wl.to_host(out, g.dtype)
    if g.dtype == "f32":
        np.testing.assert_allclose(got, ref, rtol=1e-5, atol=1e-6)
    else:
        same = got == ref
        assert same.mean() > 0.99
        step = np.abs(got.astype(np.int32) - ref.astype(np.int32))
        assert step.max() <= 1                                  # adjacent bf16 bit patterns


def test_compress_then_insert_then_attend_streams_like_the_oracle():
    """Config-5 style step with compress-on-insert: full-width new K/V -> codes -> fused step."""
    from gpu_harness import dev_storage
    g = wl.Geometry(B=3, Hq=4, Hkv=4, D=128, E=8, S=40, k=2, dtype="bf16", rank=32)
    case = wl.make_host_case(g, seed=61, utility0="exp")
    ensure_route_margin(case, g.k)
    rng = np.random.default_rng(5)
    WK = wl.encode(rng.standard_normal((g.Hkv, g.rank, g.D)) / np.sqrt(g.D), "bf16")
    WV = wl.encode(rng.standard_normal((g.Hkv, g.rank, g.D)) / np.sqrt(g.D), "bf16")
    kfull = wl.encode(rng.standard_normal((g.B, g.Hkv, g.D)), "bf16")
    vfull = wl.encode(rng.standard_normal((g.B, g.Hkv, g.D)), "bf16")
    dc = DeviceCase(case)
    kc = torch.zeros((g.B, g.Hkv, g.rank), device=DEV, dtype=torch.bfloat16)
    vc = torch.zeros_like(kc)
    pk.pikv_compress(dc.desc, dev_storage(kfull, "bf16"), dev_storage(WK, "bf16"), kc,
                     dev_storage(vfull, "bf16"), dev_storage(WV, "bf16"), vc)
    np.testing.assert_array_equal(np.abs(wl.to_host(vc, "bf16").astype(np.int32) -
                                         orc.compress(vfull, WV, dtype="bf16").astype(np.int32)) <= 1, True)
    ei = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
    ec = torch.zeros((g.B, g.E), device=DEV, dtype=torch.int32)
    pk.pikv_decode_step(dc.desc, dc.q, dc.W_r, dc.bias, kc, vc, dc.K_tab, dc.V_tab, dc.U_K, dc.U_V,
                        dc.n_valid, dc.utility, g.k, pk.COMBINE_LSE, 0.0, 1.0, dc.topk, dc.gates, ei, ec,
                        dc.y, dc.row_max, dc.row_norm, dc.scores, dc.slot_coef, dc.workspace)
    torch.cuda.synchronize()
    # oracle on the GPU's own codes (the codes themselves are checked in test_compress_matches_oracle)
    kc_h, vc_h = wl.to_host(kc, "bf16"), wl.to_host(vc, "bf16")
    ref = case.clone()
    x = np.ascontiguousarray(case.q.reshape(g.route_rows, g.d_r))
    idx, gates, _ = orc.route(x, ref.W_r, g.k, dtype=g.dtype)
    np.testing.assert_array_equal(t2n(dc.topk), idx)
    mask = np.zeros((g.B, g.E), np.int32)
    for b in range(g.B):
        mask[b, idx[b]] = 1
    ridx, rcnt = orc.evict(ref.utility, ref.n_valid, g.S - 1, shard_mask=mask, max_evict=1)
    orc.append(kc_h, vc_h, idx, ref.K_shards, ref.V_shards, ref.utility, ref.n_valid, dtype="bf16",
               reuse_idx=ridx, reuse_cnt=rcnt)
    out = oracle_step(ref, idx, gates, orc.COMBINE_LSE, utility=ref.utility, decay=1.0)
    ok, emax, l2 = y_tolerance_ok(t2n(dc.y), out["y"], g.dtype)
    assert ok, (emax, l2)
    assert_utility_close(t2n(dc.utility), ref.utility)
    for s in range(g.B * g.E):
        np.testing.assert_array_equal(dc.shard_host("K", s), ref.K_shards[s])


def test_strided_shards_on_the_matrix_core_kernel_and_the_fused_step():
    """Rows padded to a larger pitch and extra slots per head (stride_s > width, stride_h > S*stride_s)
    through the grouped-query MFMA kernel, both via the separate calls and the fused step."""
    g = wl.Geometry(B=2, Hq=8, Hkv=2, D=128, E=8, S=150, k=2, dtype="bf16")
    case = wl.make_host_case(g, seed=71, n_valid="ragged", utility0="exp")
    case.n_valid[case.n_valid == g.S] = g.S - 1
    ensure_route_margin(case, g.k)
    x = np.ascontiguousarray(case.q.reshape(g.route_rows, g.d_r))
    idx, gates, _ = orc.route(x, case.W_r, g.k, dtype=g.dtype)
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE, utility=u_ref, decay=0.5)
    for fused in (False, True):
        dc = DeviceCase(case, stride_pad=(16, 7))
        if fused:
            pk.pikv_decode_step(dc.desc, dc.q, dc.W_r, dc.bias, None, None, dc.K_tab, dc.V_tab, None, None,
                                dc.n_valid, dc.utility, g.k, pk.COMBINE_LSE, 0.0, 0.5, dc.topk, dc.gates,
                                None, None, dc.y, dc.row_max, dc.row_norm, dc.scores, dc.slot_coef,
                                dc.workspace)
        else:
            dc.route()
            dc.attend()
            dc.update_utility(0.5)
        np.testing.assert_array_equal(t2n(dc.topk), idx)
        ok, emax, l2 = y_tolerance_ok(t2n(dc.y), ref["y"], g.dtype)
        assert ok, (fused, emax, l2)
        assert_utility_close(t2n(dc.utility), u_ref)


@pytest.mark.parametrize("spec", [
    dict(B=1, Hq=128, Hkv=8, D=128, E=8, S=700, k=4, dtype="bf16"),                    # 16 rows per kv head
    dict(B=2, Hq=256, Hkv=8, D=128, E=8, S=300, k=3, dtype="bf16", tq=8),             # token-major drafts
    dict(B=1, Hq=96, Hkv=96, D=64, E=8, S=120, k=5, dtype="bf16"),                     # plain-ALU kernel
    dict(B=1, Hq=40, Hkv=8, D=32, E=4, S=90, k=2, dtype="f32", rank=16),
], ids=["gqa16_512pairs", "tq8_768pairs", "g1_480pairs", "f32_80pairs"])
@pytest.mark.parametrize("combine", [orc.COMBINE_LSE, orc.COMBINE_LOCAL], ids=["lse", "local"])
def test_fused_step_with_many_head_shard_pairs_equals_separate_calls(spec, combine):
    """More (head, shard) pairs than a utility block has groups of eight lanes: its statistics
    come from one thread per pair, and with many heads per thread the utility blocks are
    dispatched ahead of the merge blocks.  Same bits as the separate calls, two steps in a row."""
    from gpu_harness import dev_storage
    token_major = "tq" in spec
    g = wl.Geometry(token_major=token_major, **spec)
    case = wl.make_host_case(g, seed=77, n_valid="ragged", utility0="exp", w_sigma=0.02)
    ensure_route_margin(case, g.k)
    dA, dB = DeviceCase(case), DeviceCase(case)
    if token_major:
        for d in (dA, dB):
            d.desc = pk.make_desc(g.B, g.Hq, g.Hkv, g.D, g.E, g.S, dtype=pk.binding.BF16, stride_h=d.stride_h,
                                  stride_s=d.stride_s, tq=g.tq)
    eiA = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
    ecA = torch.full((g.B, g.E), -5, device=DEV, dtype=torch.int32)
    eiB, ecB = eiA.clone(), ecA.clone()
    for step in range(2):
        kn, vn = wl.draw_new_kv(g, 500 + step)
        dkn, dvn = dev_storage(kn, g.dtype), dev_storage(vn, g.dtype)
        pk.pikv_decode_step(dA.desc, dA.q, dA.W_r, dA.bias, dkn, dvn, dA.K_tab, dA.V_tab, dA.U_K, dA.U_V,
                            dA.n_valid, dA.utility, g.k, combine, 0.0, 0.9, dA.topk, dA.gates,
                            eiA, ecA, dA.y, dA.row_max, dA.row_norm, dA.scores, dA.slot_coef, dA.workspace)
        dB.route()
        pk.pikv_evict(dB.desc, dB.utility, dB.n_valid, g.S - 1, dB.topk, g.k, eiB, ecB, 1, False, None, None)
        pk.pikv_append(dB.desc, dkn, dvn, dB.topk, g.k, eiB, ecB, 1, dB.K_tab, dB.V_tab, dB.utility, dB.n_valid)
        dB.attend(combine=combine)
        dB.update_utility(0.9)
        for name in ("topk", "gates", "n_valid", "utility", "y", "row_max", "row_norm", "slot_coef"):
            np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)),
                                          err_msg="%s differs at step %d" % (name, step))


@pytest.mark.parametrize("spec", [
    dict(B=9, Hq=5, Hkv=5, D=16, E=8, S=2052, k=8, dtype="bf16"),       # four slots per thread, one tile per block
    dict(B=9, Hq=5, Hkv=5, D=16, E=8, S=2051, k=8, dtype="bf16"),       # odd capacity: one slot per thread
    dict(B=32, Hq=38, Hkv=1, D=16, E=8, S=2500, k=4, dtype="bf16"),     # several tiles of four slots, 10 heads a thread
    dict(B=4, Hq=80, Hkv=1, D=16, E=8, S=4100, k=4, dtype="f32"),       # many (head, shard) pairs
    dict(B=4, Hq=2, Hkv=1, D=128, E=8, S=2304, k=8, dtype="bf16"),      # blocks of 1024 threads
], ids=["wide", "odd", "multi", "many", "threads1024"])
def test_fused_step_on_many_slots_equals_separate_calls(spec):
    """More than one round of utility blocks: four slots per thread, against the stand-alone utility
    kernel with its access bookkeeping, bit for bit; entry counts from a few slots to full."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=5, n_valid="ragged", utility0="exp", w_sigma=0.1)
    case.n_valid[0, :4] = [3, 255, 257, g.S]
    dA, dB = DeviceCase(case), DeviceCase(case)
    for d in (dA, dB):
        d.last = torch.zeros((g.B, g.E, g.S), device=DEV, dtype=torch.int32)
        d.freq, d.birth = d.last.clone(), d.last.clone()
        d.eidx = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
        d.ecnt = torch.full((g.B, g.E), -5, device=DEV, dtype=torch.int32)
    for step in range(2):
        kn, vn = wl.draw_new_kv(g, 600 + step)
        dkn, dvn = dev_storage(kn, g.dtype), dev_storage(vn, g.dtype)
        args = pk.make_policy_args(pk.POLICY_H2O, 7 + step, threshold=2.0 / g.S, birth=dA.birth, last_access=dA.last,
                                   freq=dA.freq)
        pk.pikv_decode_step_policy(dA.desc, dA.q, dA.W_r, dA.bias, dkn, dvn, dA.K_tab, dA.V_tab, None, None, dA.n_valid,
                                   dA.utility, g.k, pk.COMBINE_LSE, 0.0, 0.9, dA.topk, dA.gates, dA.eidx, dA.ecnt, dA.y,
                                   dA.row_max, dA.row_norm, dA.scores, dA.slot_coef, dA.workspace, args)
        dB.route()
        pk.pikv_evict(dB.desc, dB.utility, dB.n_valid, g.S - 1, dB.topk, g.k, dB.eidx, dB.ecnt, 1, False, None, None)
        pk.pikv_policy_stamp(dB.desc, dB.topk, g.k, dB.eidx, dB.ecnt, 1, dB.n_valid, 7 + step, dB.birth, dB.last, dB.freq)
        pk.pikv_append(dB.desc, dkn, dvn, dB.topk, g.k, dB.eidx, dB.ecnt, 1, dB.K_tab, dB.V_tab, dB.utility, dB.n_valid)
        dB.attend()
        pk.pikv_update_utility_tracked(dB.desc, dB.scores, dB.slot_coef, dB.n_valid, dB.topk, g.k, 0.9, dB.utility,
                                       2.0 / g.S, 7 + step, dB.last, dB.freq)
        for name in ("topk", "n_valid", "utility", "y", "row_norm", "last", "freq", "birth"):
            np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)),
                                          err_msg="%s differs at step %d" % (name, step))
    assert (t2n(dA.freq) > 0).any()


def test_fused_step_with_many_heads_times_shards_uses_the_separate_merge():
    """Hq * k beyond what a utility block restages: the step falls back to separate merge and
    utility launches and still equals the separate calls bit for bit."""
    g = wl.Geometry(B=1, Hq=64, Hkv=64, D=16, E=64, S=24, k=40, dtype="bf16")
    case = wl.make_host_case(g, seed=72, utility0="exp", w_sigma=0.2)
    ensure_route_margin(case, g.k, margin=1e-4)
    dA, dB = DeviceCase(case), DeviceCase(case)
    pk.pikv_decode_step(dA.desc, dA.q, dA.W_r, dA.bias, None, None, dA.K_tab, dA.V_tab, None, None,
                        dA.n_valid, dA.utility, g.k, pk.COMBINE_LSE, 0.0, 1.0, dA.topk, dA.gates,
                        None, None, dA.y, dA.row_max, dA.row_norm, dA.scores, dA.slot_coef, dA.workspace)
    dB.route()
    dB.attend()
    dB.update_utility(1.0)
    for name in ("topk", "y", "utility"):
        np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)))
    x = np.ascontiguousarray(case.q.reshape(g.route_rows, g.d_r))
    idx, gates, _ = orc.route(x, case.W_r, g.k, dtype=g.dtype)
    np.testing.assert_array_equal(t2n(dA.topk), idx)
    u_ref = case.utility.copy()
    ref = oracle_step(case, idx, gates, orc.COMBINE_LSE, utility=u_ref)
    ok, emax, l2 = y_tolerance_ok(t2n(dA.y), ref["y"], g.dtype)
    assert ok, (emax, l2)
    assert_utility_close(t2n(dA.utility), u_ref)


# ------------------------------------------------------------------- HIP graph replay
@pytest.mark.parametrize("spec", [
    dict(B=2, Hq=8, Hkv=2, D=128, E=8, S=96, k=2, dtype="bf16"),            # matrix-core kernel
    dict(B=3, Hq=4, Hkv=4, D=64, E=8, S=80, k=3, dtype="bf16", rank=16),   # plain-ALU kernel, codes
], ids=["gqa4_d128", "rank16"])
def test_graph_replays_of_the_fused_step_equal_eager_steps(spec):
    """The benchmark times a captured graph of fused steps.  Every replay must leave exactly the
    state the same number of eager steps leaves (the step carries state: utilities, entry counts,
    evicted rows), with eager work and synchronisations of the program's own between replays."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=101, utility0="exp", zipf_s=1.1)
    kn, vn = wl.draw_new_kv(g, 102)
    per_graph, replays = 3, 4

    def run(dc, ei, ec, dkn, dvn):
        pk.pikv_decode_step(dc.desc, dc.q, dc.W_r, dc.bias, dkn, dvn, dc.K_tab, dc.V_tab, dc.U_K, dc.U_V,
                            dc.n_valid, dc.utility, g.k, pk.COMBINE_LSE, 0.0, 0.9, dc.topk, dc.gates, ei, ec,
                            dc.y, dc.row_max, dc.row_norm, dc.scores, dc.slot_coef, dc.workspace)

    def fresh():
        dc = DeviceCase(case)
        ei = torch.full((g.B, g.E, 1), -1, device=DEV, dtype=torch.int32)
        ec = torch.zeros((g.B, g.E), device=DEV, dtype=torch.int32)
        return dc, ei, ec, dev_storage(kn, g.dtype), dev_storage(vn, g.dtype)

    # eager reference trajectory, a snapshot after every per_graph steps
    dE = fresh()
    snaps = []
    for r in range(replays + 1):                  # +1: the capture pass itself executes nothing, warm-up does
        for _ in range(per_graph):
            run(*dE)
        snaps.append([t2n(x).copy() for x in (dE[0].utility, dE[0].n_valid, dE[0].y, dE[0].topk, dE[2])])

    dG = fresh()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for _ in range(per_graph):                # warm-up = the first per_graph steps of the trajectory
            run(*dG)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(per_graph):
                run(*dG)
        for r in range(replays):
            graph.replay()
            stream.synchronize()
            got = [t2n(x) for x in (dG[0].utility, dG[0].n_valid, dG[0].y, dG[0].topk, dG[2])]
            for a, b2, nm in zip(got, snaps[r + 1], ("utility", "n_valid", "y", "topk", "evicted_cnt")):
                np.testing.assert_array_equal(a, b2, err_msg="%s differs after replay %d" % (nm, r))
            # eager work of the program's own between replays (must not disturb the captured launches)
            scratch = torch.rand(1 << 16, device=DEV)
            assert float((scratch * 2).sum().item()) > 0


@pytest.mark.parametrize("spec", [
    dict(B=1, Hq=4, Hkv=2, D=128, E=3, S=400, k=2, dtype="bf16"),            # matrix-core kernel
    dict(B=2, Hq=2, Hkv=2, D=64, E=3, S=300, k=2, dtype="bf16"),             # plain-ALU kernel
    dict(B=1, Hq=2, Hkv=2, D=64, E=2, S=200, k=2, dtype="f32", rank=16),
], ids=["gqa2_d128", "g1_d64", "f32_rank16"])
def test_attention_with_very_peaked_scores(spec):
    """Scores in the hundreds (scale 8 on N(0,1) data): the softmax is a near one-hot, every
    exponent but a few underflows; nothing may overflow or lose the dominant entry.

    Tolerance: a probability is coef * exp(s - M) with s and M computed in fp32.  A score of
    magnitude |s| carries an absolute error of a few units in its last place (a 128-term fp32 dot
    product times the scale: at most 4 ulp here), so exp(s - M) carries that as a RELATIVE error,
    twice (s and M).  The utility bar of rel 1e-4 therefore widens by 8 ulp32(max |M|) - for
    |M| ~ 300 that is 2.4e-4 - and the row maximum itself is good to 4 ulp32(|M|)."""
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=23, n_valid="ragged", utility0="exp")
    idx, gates = random_selection(g, 24)
    for combine in (orc.COMBINE_LSE, orc.COMBINE_LOCAL):
        u_ref = case.utility.copy()
        ref = oracle_step(case, idx, gates, combine, utility=u_ref, decay=1.0, scale=8.0)
        dc = DeviceCase(case)
        d_idx, d_gates = torch.from_numpy(idx).to(DEV), torch.from_numpy(gates).to(DEV)
        dc.attend(topk=d_idx, gates=d_gates, combine=combine, scale=8.0)
        dc.update_utility(1.0, topk=d_idx)
        y = t2n(dc.y)
        assert np.isfinite(y).all()
        ok, emax, l2 = y_tolerance_ok(y, ref["y"], g.dtype)
        assert ok, (combine, emax, l2)
        ulp = float(np.spacing(np.float32(np.abs(ref["row_max"][np.isfinite(ref["row_max"])]).max())))
        np.testing.assert_allclose(t2n(dc.row_max), ref["row_max"], rtol=0, atol=4 * ulp)
        u = t2n(dc.utility)
        assert np.isfinite(u).all()
        np.testing.assert_allclose(u, u_ref, rtol=1e-4 + 8 * ulp, atol=1e-9)


def test_stream_read_probe_folds_every_word_once():
    """The measurement kernel behind bench.py's read-ceiling figure reads every byte it is given
    exactly once: its per-span xor of 32-bit words equals numpy's, for spans with ragged ends."""
    rng = np.random.default_rng(3)
    for n, words, parts in ((3, 70000, 5), (1, 4, 1), (2, 1024 * 37 + 12, 7), (4, 16384 * 4, 4)):
        host = rng.integers(0, 2 ** 32, size=(n, words), dtype=np.uint64).astype(np.uint32)
        bufs = [torch.from_numpy(host[i].view(np.int32).copy()).to(DEV) for i in range(n)]
        table = pk.shard_table(bufs)
        out = torch.zeros(n * parts, device=DEV, dtype=torch.int32)
        pk.pikv_stream_read_probe(table, n, words * 4, parts, out)
        got = t2n(out).view(np.uint32).reshape(n, parts)
        span = -(-(words * 4) // parts)
        span = -(-span // 4096) * 4096 // 4
        for i in range(n):
            for pt in range(parts):
                want = np.bitwise_xor.reduce(host[i, pt * span:(pt + 1) * span]) if pt * span < words else 0
                assert got[i, pt] == want, (n, words, parts, i, pt)


@pytest.mark.parametrize("spec,splits,shift", [
    (dict(B=2, Hq=7, Hkv=7, D=64, E=8, S=288, k=1, dtype="f32"), (1, 9, 32), 0),
    (dict(B=1, Hq=6, Hkv=2, D=128, E=8, S=288, k=3, dtype="bf16"), (1, 8, 9), 0),
    (dict(B=2, Hq=33, Hkv=11, D=16, E=8, S=160, k=5, dtype="f32"), (1, 5, 7), 0),
    (dict(B=1, Hq=40, Hkv=8, D=64, E=9, S=160, k=8, dtype="bf16"), (2, 4, 5), 0),
    (dict(B=1, Hq=5, Hkv=5, D=32, E=12, S=160, k=9, dtype="f32"), (1, 3, 5), 0),
    (dict(B=2, Hq=3, Hkv=3, D=128, E=4, S=1200, k=2, dtype="f32"), (33, 40), 0),
    (dict(B=2, Hq=8, Hkv=2, D=128, E=8, S=160, k=4, dtype="bf16", rank=32), (1, 3, 9), 0),
    (dict(B=2, Hq=8, Hkv=2, D=128, E=8, S=160, k=4, dtype="bf16", rank=64), (2,), 3),
    (dict(B=1, Hq=4, Hkv=4, D=32, E=8, S=160, k=2, dtype="bf16", rank=16), (2,), 0),
    (dict(B=1, Hq=4, Hkv=4, D=128, E=8, S=160, k=2, dtype="f32", rank=64), (2,), 0),
    (dict(B=1, Hq=4, Hkv=4, D=128, E=8, S=160, k=2, dtype="f32", rank=32), (2, 17), 1),
], ids=["k1", "k3", "k5", "k8", "k9", "long", "r32", "r64_shifted", "r16", "f32_r64", "f32_r32_shifted"])
def test_merge_of_every_count_of_shards_and_partials(spec, splits, shift):
    """The merge by single waves (up to eight shards) and by the block, one to four pairs a lane and more, decoders in LDS,
    too large for it and not aligned for it; y and utilities against the oracle, the fused step bit for bit
    against the separate calls."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=31, n_valid="ragged", utility0="exp", w_sigma=0.05)
    case.n_valid[0, :2] = [0, g.S]
    ensure_route_margin(case, g.k)
    for n in splits:
        pk.pikv_set_attn_split(n)
        try:
            dA, dB = DeviceCase(case), DeviceCase(case)
            if shift:                # the decoder some values into its buffer
                for d in (dA, dB):
                    d.U_V = torch.cat([d.U_V.new_zeros(shift), d.U_V.flatten()])[shift:].view(d.U_V.shape)
                    assert d.U_V.data_ptr() % 16
            idx, gates = (lambda d: (d.route(), (t2n(d.topk), t2n(d.gates)))[1])(dB)
            u_ref = case.utility.copy()
            ref = oracle_step(case, idx, gates, orc.COMBINE_LSE, utility=u_ref, decay=0.9)
            pk.pikv_decode_step(dA.desc, dA.q, dA.W_r, dA.bias, None, None, dA.K_tab, dA.V_tab, dA.U_K, dA.U_V, dA.n_valid,
                                dA.utility, g.k, pk.COMBINE_LSE, 0.0, 0.9, dA.topk, dA.gates, None, None, dA.y, dA.row_max,
                                dA.row_norm, dA.scores, dA.slot_coef, dA.workspace)
            dB.attend()
            dB.update_utility(0.9)
        finally:
            pk.pikv_set_attn_split(0)
        ok, emax, l2 = y_tolerance_ok(t2n(dB.y), ref["y"], g.dtype)
        assert ok, (n, emax, l2)
        assert_utility_close(t2n(dB.utility), u_ref)
        for name in ("topk", "gates", "utility", "y", "row_max", "row_norm", "slot_coef"):
            np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)), err_msg="%s, %d splits" % (name, n))


@pytest.mark.parametrize("spec", [
    dict(B=1, Hq=3, Hkv=3, D=16, E=4, S=63, k=2, dtype="f32", per_head_routing=True),       # fewer heads than quarters
    dict(B=2, Hq=9, Hkv=9, D=16, E=8, S=65, k=5, dtype="f32", per_head_routing=True),
    dict(B=6, Hq=9, Hkv=9, D=16, E=8, S=2051, k=3, dtype="bf16", per_head_routing=True),     # four slots, 64 apart
    dict(B=6, Hq=5, Hkv=5, D=16, E=8, S=2052, k=3, dtype="bf16", per_head_routing=True),     # four slots in a line
    dict(B=1, Hq=70, Hkv=10, D=16, E=6, S=300, k=1, dtype="f32"),                            # several batches of heads
    dict(B=12, Hq=8, Hkv=8, D=16, E=4, S=3001, k=2, dtype="bf16"),
    dict(B=12, Hq=40, Hkv=8, D=16, E=4, S=3004, k=2, dtype="bf16"),
], ids=["ph3", "ph9", "ph_apart", "ph_line", "heads70", "apart", "line"])
def test_utility_update_of_every_form(spec):
    """Per-token and head-by-head selections, one slot per thread and four, aligned rows and others, with and without the access
    bookkeeping: utilities against the oracle, slots past the count and shards nobody selected untouched."""
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=8, n_valid="ragged", utility0="exp", w_sigma=0.4)
    case.n_valid[0, :2] = [1, g.S]
    ensure_route_margin(case, g.k)
    dc = DeviceCase(case)
    dc.route()
    dc.attend()
    u_ref = case.utility.copy()
    ref = oracle_step(case, t2n(dc.topk), t2n(dc.gates), orc.COMBINE_LSE, utility=u_ref, decay=0.9)
    assert y_tolerance_ok(t2n(dc.y), ref["y"], g.dtype)[0]
    before = dc.utility.clone()
    dc.update_utility(0.9)
    got = t2n(dc.utility)
    assert_utility_close(got, u_ref)
    np.testing.assert_array_equal(got[u_ref == case.utility], case.utility[u_ref == case.utility])
    last, freq = (torch.zeros((g.B, g.E, g.S), device=DEV, dtype=torch.int32) for _ in range(2))
    threshold = 2.0 / g.S
    pk.pikv_update_utility_tracked(dc.desc, dc.scores, dc.slot_coef, dc.n_valid, dc.topk, g.k, 0.9, before, threshold, 7, last, freq)
    np.testing.assert_array_equal(t2n(before), got)
    mass = u_ref - 0.9 * case.utility * (u_ref != case.utility)      # only clear cases: the sum is rounded differently here
    touched = u_ref != case.utility
    assert (t2n(freq)[touched & (mass > 1.01 * threshold)] == 1).all()
    assert (t2n(freq)[~touched | (mass < 0.99 * threshold)] == 0).all()
    np.testing.assert_array_equal(t2n(last), 7 * t2n(freq))
    only = (torch.zeros_like(last), torch.zeros_like(freq))
    pk.pikv_update_utility_tracked(dc.desc, dc.scores, dc.slot_coef, dc.n_valid, dc.topk, g.k, 0.9, None, threshold, 7, *only)
    np.testing.assert_array_equal(t2n(only[1]), t2n(freq))


def test_the_binding_takes_what_it_took_and_refuses_what_it_refused():
    """Ordinary arguments go through the extension; numbers of other types, parameters and other streams give the same; tensors on the host,
    strided tensors and wrong types are refused as before."""
    g = wl.Geometry(B=2, Hq=4, Hkv=2, D=32, E=4, S=64, k=2, dtype="f32")
    case = wl.make_host_case(g, seed=4, w_sigma=0.3)
    dc = DeviceCase(case)
    out = []

    def route(x, W, rows=g.B, k=g.k, stream=None):
        topk, gates = torch.zeros((g.B, g.k), device=DEV, dtype=torch.int32), torch.zeros((g.B, g.k), device=DEV)
        if stream is not None:
            stream.wait_stream(torch.cuda.current_stream())           # (behind the two fills)
        pk.pikv_route(x, W, None, rows, g.d_r, g.E, k, topk, gates, stream=stream)
        out.append((t2n(topk), t2n(gates)))

    x = dc.q.reshape(g.B, -1)
    assert pk.binding._calls().pikv_route(x, dc.W_r, None, g.B, g.d_r, g.E, g.k, dc.topk, dc.gates, None, None) == 0
    route(x, dc.W_r)
    route(torch.nn.Parameter(x), dc.W_r)
    assert pk.binding._calls().pikv_route(x, dc.W_r, None, g.B, g.d_r, g.E, 2.0, dc.topk, dc.gates, None, None) is None

    class Marked(torch.Tensor):
        pass

    route(x.as_subclass(Marked), dc.W_r)
    other = torch.cuda.Stream()
    route(x, dc.W_r, stream=other)
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        route(x, dc.W_r)
        torch.cuda.current_stream().synchronize()
    other.synchronize()
    route(x, dc.W_r, k=True + 1)
    route(x, dc.W_r, rows=g.B + (1 << 32))                    # ctypes keeps the low 32 bits
    for topk, gates in out[1:]:
        np.testing.assert_array_equal(topk, out[0][0])
        np.testing.assert_array_equal(gates, out[0][1])
    with pytest.raises(ValueError, match="device memory"):
        route(x.cpu(), dc.W_r)
    with pytest.raises(ValueError, match="contiguous"):
        route(x, dc.W_r.t().contiguous().t())
    with pytest.raises(TypeError, match="storage dtype"):
        route(x.double(), dc.W_r)
    with pytest.raises(AttributeError):
        route(None, dc.W_r)
    with pytest.raises(Exception):
        route(x, dc.W_r, k=2.0)
    with pytest.raises(pk.PikvError):
        route(x, dc.W_r, k=g.E + 1)
    with pytest.raises(pk.PikvError):                         # no workspace
        pk.pikv_sharded_attn(dc.desc, dc.q, dc.K_tab, dc.V_tab, None, None, dc.n_valid, dc.topk, dc.gates, g.k, 0, 0.0, dc.y,
                             None, None, None, None, None)


@pytest.mark.parametrize("spec", [
    dict(B=2, Hq=128, Hkv=8, D=128, E=8, S=300, k=3, dtype="bf16"),      # merge by 256 threads
    dict(B=1, Hq=96, Hkv=8, D=128, E=8, S=2100, k=2, dtype="bf16"),      # by 1024, for its heads
    dict(B=3, Hq=64, Hkv=8, D=64, E=8, S=300, k=4, dtype="f32"),         # at the line: one launch
    dict(B=3, Hq=65, Hkv=5, D=64, E=8, S=300, k=4, dtype="f32"),         # past it
], ids=["256", "1024", "line", "past"])
def test_fused_step_with_feedback_on_both_sides_of_the_separate_merge(spec):
    """The router's penalty update rides with the merge where that is a launch of its own; the same bits as the separate calls."""
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=12, n_valid="ragged", utility0="exp", w_sigma=0.05)
    ensure_route_margin(case, g.k)
    dA, dB = DeviceCase(case), DeviceCase(case)
    for d in (dA, dB):
        d.load = torch.arange(g.E, device=DEV, dtype=torch.int32)
        d.after = torch.zeros(g.E, device=DEV)
    feedback = pk.make_router_feedback(pk.PENALTY_LOAD_BALANCE, 0.01, dA.load, dA.after)
    pk.pikv_decode_step_policy(dA.desc, dA.q, dA.W_r, dA.bias, None, None, dA.K_tab, dA.V_tab, None, None, dA.n_valid, dA.utility,
                               g.k, pk.COMBINE_LSE, 0.0, 0.9, dA.topk, dA.gates, None, None, dA.y, dA.row_max, dA.row_norm,
                               dA.scores, dA.slot_coef, dA.workspace, None, feedback=feedback)
    dB.route()
    dB.attend()
    dB.update_utility(0.9)
    pk.pikv_router_penalty(pk.PENALTY_LOAD_BALANCE, dB.topk, g.B, g.k, g.E, dB.load, None, 0.01, dB.after)
    for name in ("topk", "gates", "utility", "y", "row_max", "row_norm", "slot_coef", "load", "after"):
        np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)), err_msg=name)
    assert t2n(dA.load).sum() == g.E * (g.E - 1) // 2 + g.B * g.k


@pytest.mark.parametrize("spec,tile", [
    (dict(B=1, Hq=4, Hkv=4, D=64, E=4, S=256, k=2, dtype="f32", per_head_routing=True), 32),       # 16 splits of a head
    (dict(B=1, Hq=6, Hkv=2, D=64, E=12, S=32, k=12, dtype="f32", per_head_routing=True), 32),      # more shards than a wave holds
    (dict(B=1, Hq=3, Hkv=3, D=128, E=6, S=81, k=2, dtype="bf16"), 32),                             # a last tile of 17 rows
    (dict(B=1, Hq=2, Hkv=2, D=128, E=6, S=65, k=1, dtype="f32"), 16),                              # odd score rows
    (dict(B=9, Hq=7, Hkv=7, D=16, E=8, S=128, k=3, dtype="bf16"), 128),                            # a tile per shard, many heads
    (dict(B=2, Hq=2, Hkv=2, D=32, E=5, S=90, k=1, dtype="bf16"), 64),                              # fewer splits than merging waves
], ids=lambda v: str(v) if isinstance(v, int) else "D%d_S%d_k%d_%s" % (v["D"], v["S"], v["k"], v["dtype"]))
@pytest.mark.parametrize("combine", [orc.COMBINE_LSE, orc.COMBINE_LOCAL], ids=["lse", "local"])
def test_smallest_calls_in_one_launch_equal_pass_and_merge(spec, tile, combine):
    """A head per block, merge included, against the two kernels with the same splits forced: shards that hold nothing, one
    entry, part of a tile and all of it, padded strides, a query that is not 16-byte aligned, infinite values; same bits."""
    g = wl.Geometry(**spec)
    nv = np.resize(np.array([0, 1, tile - 1, tile, tile + 1, g.S - 1, g.S], np.int32), (g.B, g.E)).clip(0, g.S)
    case = wl.make_host_case(g, seed=91, n_valid=nv, utility0="exp")
    inf, ninf = (np.inf, -np.inf) if g.dtype == "f32" else (0x7f80, 0xff80)      # (bf16 as bits)
    case.V_shards[2][0, 0, 0] = inf
    case.K_shards[3][0, :2, 0] = ninf
    outs = []
    for forced in (0, (g.S + tile - 1) // tile):
        pk.pikv_set_attn_split(forced)
        try:
            dc = DeviceCase(case, stride_pad=(16, 5))
            q = torch.zeros(dc.q.numel() + 1, device=DEV, dtype=dc.q.dtype)[1:].view(dc.q.shape)
            q.copy_(dc.q)
            dc.q = q
            dc.route()
            dc.attend(combine=combine)
            outs.append({n: t2n(getattr(dc, n)).view(np.uint32) for n in ("y", "row_max", "row_norm", "slot_coef", "scores")})
            dc.attend(combine=combine, want_scores=False)
            np.testing.assert_array_equal(t2n(dc.y).view(np.uint32), outs[-1]["y"])
        finally:
            pk.pikv_set_attn_split(0)
    for name, got in outs[0].items():
        np.testing.assert_array_equal(got, outs[1][name], err_msg=name)


@pytest.mark.parametrize("spec", [
    dict(B=6, Hq=24, Hkv=8, D=16, E=6, S=2050, k=3, dtype="bf16", per_head_routing=True),     # 12 heads meet a shard; 9 tiles, the last of 2
    dict(B=5, Hq=40, Hkv=8, D=16, E=4, S=4092, k=2, dtype="bf16", per_head_routing=True),     # 20 heads; 16 tiles, aligned rows
    dict(B=2, Hq=256, Hkv=32, D=16, E=2, S=67, k=2, dtype="bf16", per_head_routing=True),     # quarters of 64 heads
    dict(B=1, Hq=130, Hkv=2, D=16, E=6, S=14000, k=1, dtype="bf16", per_head_routing=True),   # one slot per thread past 1024 blocks
    dict(B=3, Hq=130, Hkv=2, D=16, E=6, S=7420, k=1, dtype="bf16", per_head_routing=True),    # four
    dict(B=9, Hq=9, Hkv=9, D=16, E=8, S=2048, k=8, dtype="bf16"),                             # every shard, 8 tiles
], ids=["met12", "met20", "heads256", "narrow", "wide", "turned"])
def test_utility_update_by_the_heads_met_and_the_entries_held(spec):
    """Head-by-head batches of four and eight, a quarter's rows held by its lanes, shards that begin at another tile: utilities
    against the oracle over shards that hold nothing, one entry, a whole line of entries and one more, a tile's edge."""
    test_utility_update_of_every_form(spec)


@pytest.mark.parametrize("E,per_head", [(4, False), (8, True)], ids=["token", "heads"])
def test_utility_update_of_shards_that_hold_little(E, per_head):
    """Up to nine entries in shards of 4096 slots, NaN in the scores behind them: no load past the last entry's 16 bytes is needed and none
    is used; utilities of the entries against float64, the other slots as they were."""
    g = wl.Geometry(B=40, Hq=32, Hkv=8, D=16, E=E, S=4096, k=2, dtype="bf16", per_head_routing=per_head)
    rows = g.B * (g.Hq if per_head else 1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    topk = torch.rand((rows, E), device=DEV, generator=gen).argsort(1)[:, :g.k].int().contiguous()
    n_valid = torch.randint(0, 10, (g.B, E), device=DEV, generator=gen, dtype=torch.int32)
    desc = pk.make_desc(g.B, g.Hq, g.Hkv, g.D, E, g.S, dtype=1, route_rows_per_seq=g.Hq if per_head else 1)
    scores = torch.full((g.B, g.Hq, g.k, g.S), float("nan"), device=DEV)
    scores[..., :10] = torch.randn((g.B, g.Hq, g.k, 10), device=DEV, generator=gen)
    coef = torch.stack([torch.zeros((g.B, g.Hq, g.k), device=DEV),
                        torch.rand((g.B, g.Hq, g.k), device=DEV, generator=gen)], -1).contiguous()
    utility = torch.rand((g.B, E, g.S), device=DEV, generator=gen)
    want = utility.double()
    mass = torch.zeros_like(want)
    p = coef[..., 1:].double() * scores[..., :10].double().exp()
    sel = topk.long().view(g.B, -1, g.k).expand(g.B, g.Hq, g.k)
    for b in range(g.B):
        mass[b, :, :10].index_add_(0, sel[b].reshape(-1), p[b].reshape(-1, 10))
    visited = torch.zeros((g.B, E), device=DEV, dtype=torch.bool).scatter_(1, sel.reshape(g.B, -1), True)
    live = visited[..., None] & (torch.arange(g.S, device=DEV) < n_valid[..., None])
    want = torch.where(live, 0.5 * want + mass, want)
    pk.pikv_update_utility(desc, scores, coef, n_valid, topk, g.k, 0.5, utility)
    np.testing.assert_allclose(t2n(utility), t2n(want), rtol=1e-5, atol=1e-7)


def test_profile_events_bracket_the_split_pass_where_one_launch_could_merge_too():
    """The event pair stands around the kernel that streams K and V and nothing else: while it is installed a smallest call is
    the pass - which leaves its partials in the workspace - and the merge, with the same results."""
    g = wl.Geometry(B=2, Hq=4, Hkv=4, D=64, E=4, S=96, k=2, dtype="f32", per_head_routing=True)
    case = wl.make_host_case(g, seed=17, n_valid="ragged")
    dc = DeviceCase(case)
    dc.route()
    names = ("y", "row_max", "row_norm", "slot_coef")
    dc.workspace.fill_(0xa5)
    dc.attend()
    plain = {n: t2n(getattr(dc, n)) for n in names}
    assert bool((dc.workspace == 0xa5).all())                 # one launch: the workspace is not used
    start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    start.record()
    stop.record()
    pk.pikv_set_profile_events(start, stop)
    try:
        dc.attend()
        torch.cuda.synchronize()
    finally:
        pk.pikv_set_profile_events(None, None)
    assert not bool((dc.workspace == 0xa5).all())
    assert start.elapsed_time(stop) > 0
    for n in names:
        np.testing.assert_array_equal(t2n(getattr(dc, n)), plain[n], err_msg=n)


def test_every_call_of_the_extension_goes_to_the_stream_it_is_given(monkeypatch):
    """All its entry points with a stream as an argument that is being captured, another one current: nothing runs until the
    graph does, and the graph runs them all.  The ctypes path is closed meanwhile."""
    g = wl.Geometry(B=2, Hq=4, Hkv=2, D=64, E=4, S=48, k=2, dtype="f32", rank=16)
    case = wl.make_host_case(g, seed=23, n_valid="ragged", utility0="exp", w_sigma=0.3)
    case.n_valid[0, :2] = g.S
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    full = [torch.randn((g.B, g.Hkv, g.D), device=DEV, generator=gen) for _ in range(2)]
    enc = [torch.randn((g.Hkv, g.rank, g.D), device=DEV, generator=gen) / 8 for _ in range(2)]
    i32 = dict(device=DEV, dtype=torch.int32)

    def state():
        dc = DeviceCase(case)
        s = dict(dc.__dict__)
        s.update(new_K=torch.zeros((g.B, g.Hkv, g.rank), device=DEV), new_V=torch.zeros((g.B, g.Hkv, g.rank), device=DEV),
                 value=torch.zeros((g.B, g.E, g.S), device=DEV), eidx=torch.zeros((g.B, g.E, 1), **i32), ecnt=torch.zeros((g.B, g.E), **i32),
                 y2=torch.zeros_like(dc.y), load=torch.zeros(g.E, **i32), after=torch.zeros(g.E, device=DEV),
                 load2=torch.zeros(g.E, **i32), after2=torch.zeros(g.E, device=DEV),
                 first=torch.zeros((g.B, g.E, 1), **i32), one=torch.ones((g.B, g.E), **i32), left=torch.full((g.B, g.E), g.S - 1, **i32),
                 topk3=torch.zeros_like(dc.topk), topk4=torch.zeros_like(dc.topk), y3=torch.zeros_like(dc.y), y4=torch.zeros_like(dc.y))
        for name in ("birth", "last", "freq", "birth2", "last2", "freq2"):
            s[name] = (torch.arange(g.B * g.E * g.S, **i32) * 7 % 50).reshape(g.B, g.E, g.S)
        return s

    def calls(s, stream):
        d, k = s["desc"], g.k
        attn = (d, s["q"], s["K_tab"], s["V_tab"], s["U_K"], s["U_V"], s["n_valid"], s["topk"], s["gates"], k, pk.COMBINE_LSE, 0.0)
        pk.pikv_compress(d, full[0], enc[0], s["new_K"], full[1], enc[1], s["new_V"], stream=stream)
        pk.pikv_route(s["q"], s["W_r"], None, g.B, g.d_r, g.E, k, s["topk"], s["gates"], s["probs"], stream=stream)
        pk.pikv_policy_utility(d, pk.POLICY_LRU_PLUS, s["n_valid"], 60, 0.5, 0, 0, s["birth"], s["last"], s["freq"], None, s["value"],
                               stream=stream)
        pk.pikv_evict(d, s["value"], s["n_valid"], g.S - 1, s["topk"], k, s["eidx"], s["ecnt"], 1, False, None, None, stream=stream)
        pk.pikv_policy_stamp(d, s["topk"], k, s["eidx"], s["ecnt"], 1, s["n_valid"], 60, s["birth"], s["last"], s["freq"], stream=stream)
        pk.pikv_append(d, s["new_K"], s["new_V"], s["topk"], k, s["eidx"], s["ecnt"], 1, s["K_tab"], s["V_tab"], s["utility"],
                       s["n_valid"], stream=stream)
        pk.pikv_sharded_attn(*attn, s["y"], s["row_max"], s["row_norm"], s["scores"], s["slot_coef"], s["workspace"], stream=stream)
        pk.pikv_sharded_attn_noalloc(*attn, s["y2"], None, None, None, None, stream=stream)
        pk.pikv_update_utility(d, s["scores"], s["slot_coef"], s["n_valid"], s["topk"], k, 0.9, s["utility"], stream=stream)
        pk.pikv_update_utility_tracked(d, s["scores"], s["slot_coef"], s["n_valid"], s["topk"], k, 0.9, None, 0.01, 60, s["last"],
                                       s["freq"], stream=stream)
        pk.pikv_policy_compact(d, s["first"], s["one"], 1, s["left"], s["birth2"], s["last2"], s["freq2"], stream=stream)
        pk.pikv_router_penalty(pk.PENALTY_LOAD_BALANCE, s["topk"], g.B, k, g.E, s["load"], None, 0.01, s["after"], stream=stream)
        step = (d, s["q"], s["W_r"], None, None, None, s["K_tab"], s["V_tab"], s["U_K"], s["U_V"], s["n_valid"], s["utility"], k,
                pk.COMBINE_LSE, 0.0, 0.9)
        rest = (s["row_max"], s["row_norm"], s["scores"], s["slot_coef"], s["workspace"])
        pk.pikv_decode_step(*step, s["topk3"], s["gates"], None, None, s["y3"], *rest, stream=stream)
        pk.pikv_decode_step_policy(*step, s["topk4"], s["gates"], None, None, s["y4"], *rest,
                                   pk.make_policy_args(pk.POLICY_LRU, 61, threshold=0.01, birth=s["birth"], last_access=s["last"],
                                                       freq=s["freq"]),
                                   feedback=pk.make_router_feedback(pk.PENALTY_LOAD_BALANCE, 0.01, s["load2"], s["after2"]), stream=stream)

    def bits(s):
        return {n: t2n(t).view(np.uint8) for n, t in s.items() if isinstance(t, torch.Tensor) and n != "workspace" and not n.endswith("_tab")}

    eager, captured = state(), state()
    before = bits(captured)
    calls(state(), torch.cuda.current_stream())                # the kernels are loaded and the noalloc array is found
    torch.cuda.synchronize()
    graph, other, third = torch.cuda.CUDAGraph(), torch.cuda.Stream(), torch.cuda.Stream()
    assert other.cuda_stream != third.cuda_stream
    with monkeypatch.context() as m:
        m.setattr(pk.binding, "load_library", lambda: pytest.fail("a call went through ctypes"))
        with torch.cuda.graph(graph, stream=other), torch.cuda.stream(third):
            calls(captured, other)
    for name, a in bits(captured).items():
        np.testing.assert_array_equal(a, before[name], err_msg=name)
    changed = set()
    for _ in range(3):
        graph.replay()
        calls(eager, None)
        got, want = bits(captured), bits(eager)
        for name in want:
            np.testing.assert_array_equal(got[name], want[name], err_msg=name)
        changed |= {name for name in want if not np.array_equal(want[name], before[name])}
    assert {"new_K", "topk", "value", "ecnt", "birth", "K", "y", "y2", "utility", "freq", "birth2", "load", "y3", "y4", "load2"} <= changed


@pytest.mark.parametrize("spec,shift", [
    (dict(B=3, Hq=4, Hkv=2, D=128, E=4, S=160, k=2, dtype="f32", rank=32), 0),      # 16896 bytes with the row: just too large for LDS
    (dict(B=2, Hq=4, Hkv=4, D=128, E=4, S=160, k=3, dtype="f32", rank=64), 0),
    (dict(B=2, Hq=4, Hkv=4, D=64, E=4, S=160, k=2, dtype="f32", rank=64), 0),       # 16640: the largest that fits
    (dict(B=2, Hq=4, Hkv=2, D=128, E=4, S=160, k=2, dtype="bf16", rank=32), 3),     # not aligned for it
    (dict(B=2, Hq=4, Hkv=4, D=32, E=12, S=64, k=9, dtype="f32", rank=16), 1),       # weights by the whole block
], ids=["f32_r32", "f32_r64", "f32_r64_fits", "shifted", "k9_shifted"])
@pytest.mark.parametrize("splits", [1, 20], ids=["256", "1024"])
def test_additive_row_of_decoders_read_from_memory(spec, shift, splits):
    """The decoder's additive term where the merge reads the decoder where it is, by blocks of 256 and of 1024 threads (20 splits a shard), a
    sequence of empty shards among the others; y against the oracle, the fused step bit for bit against the separate calls."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    case = wl.make_host_case(g, seed=63, n_valid="ragged", utility0="exp", w_sigma=0.05)
    case.n_valid[-1, :] = 0
    ensure_route_margin(case, g.k)
    b_V = wl.encode(np.random.default_rng(64).standard_normal((g.Hkv, g.D)), g.dtype)
    rows = dev_storage(np.ascontiguousarray(np.concatenate([case.U_V, b_V[:, None, :]], axis=1)), g.dtype)
    pk.pikv_set_attn_split(splits)
    try:
        dA, dB = DeviceCase(case), DeviceCase(case)
        for d in (dA, dB):
            d.U_V = torch.cat([rows.new_zeros(shift), rows.flatten()])[shift:].view(rows.shape)
            assert (d.U_V.data_ptr() % 16 != 0) == (shift != 0)
            d.desc = pk.make_desc(g.B, g.Hq, g.Hkv, g.D, g.E, g.S, rank=g.rank, dtype=pk.binding.F32 if g.dtype == "f32" else pk.binding.BF16,
                                  stride_h=d.stride_h, stride_s=d.stride_s, flags=pk.DESC_VALUE_BIAS)
        dB.route()
        dB.attend()
        dB.update_utility(0.9)
        pk.pikv_decode_step(dA.desc, dA.q, dA.W_r, dA.bias, None, None, dA.K_tab, dA.V_tab, dA.U_K, dA.U_V, dA.n_valid, dA.utility, g.k,
                            pk.COMBINE_LSE, 0.0, 0.9, dA.topk, dA.gates, None, None, dA.y, dA.row_max, dA.row_norm, dA.scores,
                            dA.slot_coef, dA.workspace)
    finally:
        pk.pikv_set_attn_split(0)
    ref = orc.attend(case.q, case.K_shards, case.V_shards, case.n_valid, t2n(dB.topk), t2n(dB.gates), Hkv=g.Hkv, E=g.E, S=g.S,
                     dtype=g.dtype, rank=g.rank, U_K=case.U_K, U_V=case.U_V, V_bias=b_V, combine=orc.COMBINE_LSE)
    ok, emax, l2 = y_tolerance_ok(t2n(dB.y), ref["y"], g.dtype)
    assert ok, (emax, l2)
    assert (t2n(dB.y)[-1] == 0).all()
    for name in ("topk", "gates", "utility", "y", "row_max", "row_norm", "slot_coef"):
        np.testing.assert_array_equal(t2n(getattr(dA, name)), t2n(getattr(dB, name)), err_msg=name)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [16, 32, 64, 128])
@pytest.mark.parametrize("rank", [16, 32, 64])
def test_compress_of_every_form(D, rank, dtype):
    """One, two and four chunks per lane - in heads of 16 values most lanes lie past the row's end -, one pass of code elements and two, waves
    past the rank; keys and values in one launch.  The bounds are test_compress_matches_oracle's: up to 128 products, summed in another order."""
    from gpu_harness import dev_storage
    g = wl.Geometry(B=5, Hq=3, Hkv=3, D=D, E=2, S=8, k=1, dtype=dtype, rank=rank)
    rng = np.random.default_rng(10)
    desc = pk.make_desc(g.B, g.Hq, g.Hkv, D, g.E, g.S, rank=rank, dtype=pk.binding.F32 if dtype == "f32" else pk.binding.BF16)
    x = [wl.encode(rng.standard_normal((g.B, g.Hkv, D)), dtype) for _ in range(2)]
    W = [wl.encode(rng.standard_normal((g.Hkv, rank, D)) / np.sqrt(D), dtype) for _ in range(2)]
    tail = 64                                                 # values behind the codes that must stay
    out = [torch.full((g.B * g.Hkv * rank + tail,), 7.0, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16) for _ in range(2)]
    pk.pikv_compress(desc, dev_storage(x[0], dtype), dev_storage(W[0], dtype), out[0], dev_storage(x[1], dtype), dev_storage(W[1], dtype), out[1])
    for t, xs, Ws in zip(out, x, W):
        torch.cuda.synchronize()
        assert bool((t[-tail:] == 7.0).all())
        got, ref = wl.to_host(t[:-tail].view(g.B, g.Hkv, rank), dtype), orc.compress(xs, Ws, dtype=dtype)
        if dtype == "f32":
            np.testing.assert_allclose(got, ref, rtol=1e-5, atol=1e-6)
        else:
            assert (got == ref).mean() > 0.99
            assert np.abs(got.astype(np.int32) - ref.astype(np.int32)).max() <= 1


@pytest.mark.parametrize("spec,max_evict", [
    (dict(B=2, Hq=32, Hkv=32, D=128, E=64, S=9, k=5, dtype="f32"), 3),               # 1024 chunks a token: four rounds of a block
    (dict(B=3, Hq=5, Hkv=5, D=128, E=7, S=6, k=7, dtype="bf16", rank=16), 1),        # 10 chunks, every shard
    (dict(B=1, Hq=1, Hkv=1, D=16, E=1, S=4, k=1, dtype="bf16"), 2),                  # 2 chunks, one shard
], ids=["E64", "k7_rank16", "least"])
def test_append_into_freed_slots_and_behind_the_entries(spec, max_evict):
    """Every shard's count, freed slots and addresses are read ahead of the selection that picks among them: full shards, empty ones, shards
    with one free slot, with several freed slots of which the first counts, with counts the reuse list does not use; padded strides."""
    from gpu_harness import dev_storage
    g = wl.Geometry(**spec)
    rng = np.random.default_rng(77)
    case = wl.make_host_case(g, seed=78, utility0="exp")
    case.n_valid[:] = np.resize(np.array([g.S, 0, g.S - 1, 1, g.S], np.int32), (g.B, g.E))
    cnt = np.resize(np.array([0, 0, 1, max_evict], np.int32), (g.B, g.E)) * (case.n_valid > 0) * (case.n_valid < g.S)
    idx = rng.integers(0, np.maximum(case.n_valid, 1)[..., None], (g.B, g.E, max_evict)).astype(np.int32)
    idx[cnt == 0] = -5                                        # not to be used
    sel = np.stack([rng.permutation(g.E)[:g.k] for _ in range(g.B)]).astype(np.int32)
    kn, vn = wl.draw_new_kv(g, 6)
    for reuse in (True, False):
        dc = DeviceCase(case, stride_pad=(16, 2))
        want_K, want_V = dc.K.clone(), dc.V.clone()
        want_n, want_u = case.n_valid.copy(), case.utility.copy()
        new = [dev_storage(a, g.dtype) for a in (kn, vn)]
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(DEV)
        pk.pikv_append(dc.desc, new[0], new[1], up(sel), g.k, up(idx) if reuse else None, up(cnt) if reuse else None, max_evict,
                       dc.K_tab, dc.V_tab, dc.utility, dc.n_valid)
        for b in range(g.B):
            for e in sel[b]:
                n = case.n_valid[b, e]
                slot = idx[b, e, 0] if reuse and cnt[b, e] > 0 else n
                if n < g.S:
                    want_K[b * g.E + e, :, slot, :g.width] = new[0][b]
                    want_V[b * g.E + e, :, slot, :g.width] = new[1][b]
                    want_n[b, e], want_u[b, e, slot] = n + 1, 0.0
        np.testing.assert_array_equal(t2n(dc.n_valid), want_n)
        np.testing.assert_array_equal(t2n(dc.utility), want_u)
        assert torch.equal(dc.K, want_K) and torch.equal(dc.V, want_V)
