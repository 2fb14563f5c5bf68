"""Performance cases of the routed sharded-KV decode path, through the public binding.

Four kinds of pass:

  step   one fused decode step of a layer (pikv_decode_step / pikv_decode_step_policy, with
         pikv_compress in front where the cache holds rank-r codes of freshly computed K/V)
  calls  the same step as the separate calls (route, evict, append, attention, utility)
  trim   a bulk eviction with compaction: every shard is cut back to its capacity
  route  the router alone over the tokens of a prompt

With "graph" a pass replays a HIP graph of the step that was captured once, the way bench.py and
a serving loop run it; otherwise every pass makes its calls eagerly.
"""
import math

import torch

import paper_2508_06526_amd as pk

DEV = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
NOW = 1000            # step counter of the scheduling policies
PENALTY = 0.01        # load-balance coefficient

STEP = dict(kind="step", B=1, Hq=32, Hkv=8, D=128, E=16, S=4096, k=2, rank=0, dtype="bf16", per_head=False, tq=1,
            fill="full", bias=False, decay=1.0, local=False, policy="none", feedback=False, value_bias=False,
            graph=False)


def _case(name, **kw):
    return dict(STEP, name=name, **kw)


def listed():
    return [
        # the smallest model: fp32, one routing decision per (token, head), separate calls; all launches
        _case("tiny_f32_per_head", kind="calls", Hq=4, Hkv=4, D=64, E=4, S=256, per_head=True, dtype="f32"),
        # an fp32 research model of odd sizes: 6 experts (rows of W_r that are no power of two), 1501 slots
        _case("odd_f32_gqa", kind="calls", B=4, Hq=16, Hkv=4, D=64, E=6, S=1501, k=3, dtype="f32", fill="ragged",
              local=True),
        # 128K tokens of context over 16 shards, one sequence: the benchmark's workload
        _case("long_context_gqa", S=8192, k=4, bias=True, graph=True),
        # the same model early in a generation: shards of 8192 slots that hold a few hundred entries
        _case("young_cache_gqa", B=4, S=8192, k=4, bias=True, fill="short", feedback=True, graph=True),
        # speculative decoding: 8 draft tokens share every K/V load
        _case("draft8_gqa", Hq=256, S=8192, k=4, bias=True, tq=8, graph=True),
        # a serving batch of sequences of different lengths, one kv head per query head
        _case("batch_ragged_mha", B=8, Hkv=32, fill="ragged"),
        # a serving batch of a model with 64-wide heads and 8 query heads per kv head
        _case("batch_gqa_d64", B=16, Hkv=4, D=64, E=8),
        # streaming at the memory bound: every step evicts one entry per visited shard, decayed scores; the largest
        _case("streaming_mha", B=32, Hkv=32, E=8, S=2048, decay=0.9),
        # rank-32 codes, compressed on insert, one kv head per query head
        _case("codes_mha", B=16, Hkv=32, S=2048, rank=32, bias=True, graph=True),
        # rank-32 codes under grouped queries with the decoder's additive term, evicted by recency and use
        _case("codes_gqa_lru", B=16, rank=32, bias=True, policy="lru_plus", value_bias=True),
        # a memory limit lowered while serving: every shard drops a quarter of its entries and compacts
        _case("trim_compact", kind="trim", S=8192),
        # the router over a prompt
        _case("route_prompt", kind="route", B=4096, k=4, bias=True),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "calls", "calls", "trim", "route"])
    G = rng.choice([1, 1, 2, 3, 4, 4, 6, 7, 8, 8, 16])
    Hkv = rng.choice([1, 2, 4, 8, 32] if G == 1 else [1, 2, 4, 8])
    c = dict(STEP, kind=kind, Hkv=Hkv, Hq=min(128, G * Hkv) // Hkv * Hkv, D=rng.choice([64, 128, 128]),
             E=rng.choice([4, 6, 8, 8, 12, 16, 16, 16, 24, 32]), S=_logint(rng, 200, 8192),
             dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), fill=rng.choice(["full", "ragged", "ragged", "short"]),
             bias=rng.random() < 0.5, decay=rng.choice([1.0, 0.9]), local=rng.random() < 0.3)
    if rng.random() < 0.5:
        c["S"] = max(256, c["S"] // 256 * 256)
    c["k"] = rng.randint(1, min(4, c["E"]))
    if kind == "route":
        c.update(B=_logint(rng, 64, 4096), Hq=rng.choice([16, 32, 64]))
        return c
    c["B"] = _logint(rng, 1, 32)
    if kind == "step":
        c["rank"] = rng.choice([0, 0, 0, 16, 32, 64])
        c["value_bias"] = c["rank"] > 0 and rng.random() < 0.5
        c["policy"] = rng.choice(["none", "none", "lru", "lru_plus", "sl"])
        c["feedback"] = rng.random() < 0.3
        c["graph"] = rng.random() < 0.5
        if c["rank"] == 0 and c["dtype"] == "bf16" and c["D"] == 128 and 2 <= G <= 4 and rng.random() < 0.4:
            c.update(tq=4, Hq=c["Hq"] * 4)
    elif kind == "calls":
        c["per_head"] = rng.random() < 0.4
    # the cache of a state, and what a pass reads of it, stay within the largest listed case's
    while c["B"] > 1 and (_shard_bytes(c) * c["E"] * c["B"] > (8 << 30) or _shard_bytes(c) * c["k"] * c["B"] > (2 << 30)):
        c["B"] //= 2
    if _shard_bytes(c) * c["E"] * c["B"] > (8 << 30):
        c["E"] = c["k"] = 4
    return c


def _esize(c):
    return 4 if c["dtype"] == "f32" else 2


def _width(c):
    return c["rank"] or c["D"]


def _shard_bytes(c):
    return 2 * c["Hkv"] * c["S"] * _width(c) * _esize(c)


def _capacity(c):
    return max(1, c["S"] * 3 // 4)


def _d_r(c):
    return c["D"] if c["per_head"] else c["Hq"] // c["tq"] * c["D"]


def _rows(c):
    return c["B"] * (c["Hq"] if c["per_head"] else 1)


def _mean_fill(c):
    return {"full": c["S"], "ragged": c["S"] * 0.55, "short": _short(c) * 0.55}[c["fill"]]


def _short(c):
    return max(16, c["S"] // 8)


def work(case):
    """K/V rows (or codes) of the selected shards, the utilities of their entries (read and
    written), router weights, queries and outputs once; for separate attention calls the scores
    they hand to the utility update as well."""
    c = case
    es, w, S = _esize(c), _width(c), c["S"]
    if c["kind"] == "route":
        n = c["B"] * _d_r(c)
        return {"bytes": n * es + _d_r(c) * c["E"] * es + c["B"] * c["k"] * 8, "flops": 2 * n * c["E"]}
    shards = c["B"] * c["E"]
    if c["kind"] == "trim":
        kept = _capacity(c)
        return {"bytes": shards * (2 * 2 * c["Hkv"] * kept * w * es + 4 * S + 4 * kept + 4 * (S - kept)), "flops": shards * S}
    n = _mean_fill(c)
    read = _rows(c) * c["k"] if c["per_head"] else c["B"] * c["Hkv"] * c["k"]     # (kv head, shard) streams
    heads = c["B"] * c["Hq"]
    bytes_ = read * n * 2 * w * es + c["B"] * c["k"] * n * 8 + heads * c["D"] * (es + 4) + _d_r(c) * c["E"] * es
    if c["rank"]:
        bytes_ += 4 * c["Hkv"] * c["rank"] * c["D"] * es
    if c["kind"] == "calls":
        bytes_ += heads * c["k"] * n * 4
    if c["policy"] != "none":
        bytes_ += c["B"] * c["k"] * n * 8
    return {"bytes": bytes_, "flops": heads * c["k"] * n * 4 * w + 2 * _rows(c) * _d_r(c) * c["E"]}


def tolerance(case):
    """Four times what the path showed against 64 bits over these ranges, rounded up."""
    if case["kind"] == "trim":
        return "exact"
    if case["kind"] == "route":
        return {"rel": 2e-6, "max": 8e-5, "differ": 1e-3}
    return {"rel": 8e-6, "max": 3.2e-4, "differ": 1e-4}


# ------------------------------------------------------------------------------- inputs
def _empty_state(c):
    """All buffers of a pass; the cache is empty."""
    B, Hq, Hkv, D, E, S, k, w = c["B"], c["Hq"], c["Hkv"], c["D"], c["E"], c["S"], c["k"], _width(c)
    t, R = DTYPES[c["dtype"]], _rows(c)
    i32 = dict(device=DEV, dtype=torch.int32)
    s = dict(case=c, graph=None)
    s["x" if c["kind"] == "route" else "q"] = torch.zeros((B, Hq, D), device=DEV, dtype=t)
    s["W_r"] = torch.zeros((_d_r(c), E), device=DEV, dtype=t)
    s["bias"] = torch.zeros(E, device=DEV) if c["bias"] or c["feedback"] else None
    s["topk"], s["gates"] = torch.zeros((R, k), **i32), torch.zeros((R, k), device=DEV)
    if c["kind"] == "route":
        return s
    s["K"] = torch.zeros((B, E, Hkv, S, w), device=DEV, dtype=t)
    s["V"] = torch.zeros((B, E, Hkv, S, w), device=DEV, dtype=t)
    s["K_tab"], s["V_tab"] = pk.shard_table(s["K"]), pk.shard_table(s["V"])
    s["n_valid"], s["n_before"] = torch.zeros((B, E), **i32), torch.zeros((B, E), **i32)
    s["utility"] = torch.zeros((B, E, S), device=DEV)
    s["desc"] = pk.make_desc(B, Hq, Hkv, D, E, S, rank=c["rank"], dtype=0 if c["dtype"] == "f32" else 1,
                             route_rows_per_seq=Hq if c["per_head"] else 1,
                             flags=pk.DESC_VALUE_BIAS if c["value_bias"] else 0, tq=c["tq"])
    if c["kind"] == "trim":
        s["drop"] = S - _capacity(c)
        s["eidx"], s["ecnt"] = torch.zeros((B, E, s["drop"]), **i32), torch.zeros((B, E), **i32)
        s["scored"] = torch.zeros((B, E, S), device=DEV)
        return s
    s["U_K"] = s["U_V"] = None
    if c["rank"]:
        s["U_K"] = torch.zeros((Hkv, c["rank"], D), device=DEV, dtype=t)
        s["U_V"] = torch.zeros((Hkv, c["rank"] + int(c["value_bias"]), D), device=DEV, dtype=t)
        s["K_full"], s["V_full"] = (torch.zeros((B, Hkv, D), device=DEV, dtype=t) for _ in range(2))
        s["enc_K"], s["enc_V"] = (torch.zeros((Hkv, c["rank"], D), device=DEV, dtype=t) for _ in range(2))
    s["K_new"], s["V_new"] = (torch.zeros((B, Hkv, w), device=DEV, dtype=t) for _ in range(2))
    s["eidx"], s["ecnt"] = torch.zeros((B, E, 1), **i32), torch.zeros((B, E), **i32)
    s["y"] = torch.zeros((B, Hq, D), device=DEV)
    s["row_max"], s["row_norm"] = torch.zeros((B, Hq), device=DEV), torch.zeros((B, Hq), device=DEV)
    s["scores"] = torch.zeros((B, Hq, k, S), device=DEV)
    s["slot_coef"] = torch.zeros((B, Hq, k, 2), device=DEV)
    s["workspace"] = torch.empty(pk.pikv_attn_workspace_bytes(s["desc"], k), device=DEV, dtype=torch.uint8)
    if c["policy"] != "none":
        s["birth"], s["last_access"], s["freq"] = (torch.zeros((B, E, S), **i32) for _ in range(3))
    if c["feedback"]:
        s["load"] = torch.zeros(E, **i32)
    return s


def _zipf_bias(E, gen):
    order = torch.randperm(E, generator=gen, device=DEV) + 1
    p = order.double() ** -1.1
    return (p / p.sum()).log().float()


def _fill(s, seed):
    """The seeded contents: unit normal K, V, codes and queries, a router whose logits are of
    order one, utilities that are sums of probabilities."""
    c = s["case"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    B, E, S = c["B"], c["E"], c["S"]

    def normal(t, std=1.0):
        for part in (t if t.numel() > (1 << 26) else [t]):      # a large cache sequence by sequence
            part.normal_(0.0, std, generator=gen)

    normal(s["W_r"], 0.3 if c["per_head"] else 1.28 / math.sqrt(_d_r(c)))
    normal(s["x" if c["kind"] == "route" else "q"])
    if s["bias"] is not None:
        s["bias"].copy_(_zipf_bias(E, gen) if c["bias"] else torch.zeros(E, device=DEV))
    if c["kind"] == "route":
        return
    normal(s["K"])
    normal(s["V"])
    top = S if c["fill"] != "short" else _short(c)
    if c["fill"] == "full" or c["kind"] == "trim":
        s["n_valid"].fill_(S)
    else:                                # lengths between a tenth of the range and all of it
        u = torch.rand((B, E), generator=gen, device=DEV)
        s["n_valid"].copy_((top * (0.1 + 0.9 * u)).int().clamp_(1, top))
    s["n_before"].copy_(s["n_valid"])
    score = torch.empty((B, E, S), device=DEV).exponential_(1.0, generator=gen) / S
    if c["kind"] == "trim":
        s["scored"].copy_(score)
        s["utility"].zero_()
        return
    live = torch.arange(S, device=DEV) < s["n_valid"][..., None]
    s["utility"].copy_(score * live)
    for name, std in (("K_new", 1.0), ("V_new", 1.0)):
        normal(s[name], std)
    if c["rank"]:
        normal(s["U_K"], 1 / math.sqrt(c["rank"]))
        normal(s["U_V"], 1 / math.sqrt(c["rank"]))
        normal(s["K_full"])
        normal(s["V_full"])
        normal(s["enc_K"], 1 / math.sqrt(c["D"]))
        normal(s["enc_V"], 1 / math.sqrt(c["D"]))
    if c["policy"] != "none":
        s["birth"].random_(0, NOW // 2, generator=gen)
        s["last_access"].random_(NOW // 2, NOW, generator=gen)
        s["freq"].random_(0, 50, generator=gen)
    if c["feedback"]:
        s["load"].random_(0, 100, generator=gen)


def prepare(case, seed):
    s = _empty_state(case)
    if case["graph"]:
        _pass(s)                        # on the empty cache: the library and its kernels are loaded
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _pass(s)
        for name in ("topk", "gates", "eidx", "ecnt", "y", "row_max", "row_norm"):
            s[name].zero_()
    _fill(s, seed)
    if case["graph"]:
        s["graph"] = graph
    return s


# --------------------------------------------------------------------------------- passes
def _pass(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "route":
        pk.pikv_route(s["x"], s["W_r"], s["bias"], c["B"], _d_r(c), c["E"], c["k"], s["topk"], s["gates"])
    elif kind == "trim":
        s["n_valid"].copy_(s["n_before"])       # the shards have filled up and been scored again
        s["utility"].copy_(s["scored"])
        pk.pikv_evict(s["desc"], s["utility"], s["n_valid"], _capacity(c), None, 0, s["eidx"], s["ecnt"], s["drop"],
                      True, s["K_tab"], s["V_tab"])
    else:
        if c["fill"] != "full" and not c["per_head"]:
            s["n_valid"].copy_(s["n_before"])   # the token of the pass before was a rejected draft: the
        (_calls if kind == "calls" else _step)(s)                       # fill of the cache stays what it is


def _calls(s):
    c, k, d = s["case"], s["case"]["k"], s["desc"]
    pk.pikv_route(s["q"], s["W_r"], s["bias"], _rows(c), _d_r(c), c["E"], k, s["topk"], s["gates"])
    if not c["per_head"]:
        pk.pikv_evict(d, s["utility"], s["n_valid"], c["S"] - 1, s["topk"], k, s["eidx"], s["ecnt"], 1, False, None,
                      None)
        pk.pikv_append(d, s["K_new"], s["V_new"], s["topk"], k, s["eidx"], s["ecnt"], 1, s["K_tab"], s["V_tab"],
                       s["utility"], s["n_valid"])
    pk.pikv_sharded_attn(d, s["q"], s["K_tab"], s["V_tab"], s["U_K"], s["U_V"], s["n_valid"], s["topk"], s["gates"],
                         k, pk.COMBINE_LOCAL if c["local"] else pk.COMBINE_LSE, 0.0, s["y"], s["row_max"],
                         s["row_norm"], s["scores"], s["slot_coef"], s["workspace"])
    pk.pikv_update_utility(d, s["scores"], s["slot_coef"], s["n_valid"], s["topk"], k, c["decay"], s["utility"])


def _step(s):
    c, k, d = s["case"], s["case"]["k"], s["desc"]
    combine = pk.COMBINE_LOCAL if c["local"] else pk.COMBINE_LSE
    if c["rank"]:
        pk.pikv_compress(d, s["K_full"], s["enc_K"], s["K_new"], s["V_full"], s["enc_V"], s["V_new"])
    policy = feedback = None
    if c["policy"] != "none":
        policy = pk.make_policy_args({"lru": pk.POLICY_LRU, "lru_plus": pk.POLICY_LRU_PLUS, "sl": pk.POLICY_SL}[c["policy"]],
                                     NOW, lam=0.5, window=NOW * 3 // 4, threshold=1.0 / c["S"], birth=s["birth"],
                                     last_access=s["last_access"], freq=s["freq"])
    if c["feedback"]:
        feedback = pk.make_router_feedback(pk.PENALTY_LOAD_BALANCE, PENALTY, s["load"], s["bias"])
    if policy is None and feedback is None:
        pk.pikv_decode_step(d, s["q"], s["W_r"], s["bias"], s["K_new"], s["V_new"], s["K_tab"], s["V_tab"], s["U_K"],
                            s["U_V"], s["n_valid"], s["utility"], k, combine, 0.0, c["decay"], s["topk"], s["gates"],
                            s["eidx"], s["ecnt"], s["y"], s["row_max"], s["row_norm"], s["scores"], s["slot_coef"],
                            s["workspace"])
    else:
        pk.pikv_decode_step_policy(d, s["q"], s["W_r"], s["bias"], s["K_new"], s["V_new"], s["K_tab"], s["V_tab"],
                                   s["U_K"], s["U_V"], s["n_valid"], s["utility"], k, combine, 0.0, c["decay"],
                                   s["topk"], s["gates"], s["eidx"], s["ecnt"], s["y"], s["row_max"], s["row_norm"],
                                   s["scores"], s["slot_coef"], s["workspace"], policy, feedback=feedback)


def run(state):
    s = state
    if s["graph"] is not None:
        s["graph"].replay()
    else:
        _pass(s)
    return {name: s[name] for name in _outputs(s["case"])}


def _outputs(c):
    if c["kind"] == "route":
        return ["topk", "gates"]
    if c["kind"] == "trim":
        return ["K", "V", "utility", "n_valid", "eidx", "ecnt"]
    names = ["topk", "gates", "y", "row_max", "row_norm", "utility"]
    if not c["per_head"]:
        names += ["K", "V", "n_valid", "ecnt"]
    if c["rank"]:
        names += ["K_new", "V_new"]
    if c["policy"] != "none":
        names += ["birth", "last_access", "freq"]
    if c["feedback"]:
        names += ["load", "bias"]
    return names


# ---------------------------------------------------------------------------- 64-bit values
def exact(case, seed):
    c = case
    s = _empty_state(c)
    _fill(s, seed)
    out = dict.fromkeys(_outputs(c))
    B, Hq, Hkv, D, E, S, k, R = c["B"], c["Hq"], c["Hkv"], c["D"], c["E"], c["S"], c["k"], _rows(c)
    if c["kind"] == "trim":
        for b in range(B):
            for e in range(E):
                u, cap = s["scored"][b, e], _capacity(c)
                s["utility"][b, e] = u
                order = torch.argsort(u, descending=True, stable=True)
                keep, gone = order[:cap].sort().values, order[cap:].sort().values
                s["eidx"][b, e] = gone.int()
                for t in (s["K"], s["V"]):
                    t[b, e, :, :cap] = t[b, e][:, keep]
                s["utility"][b, e, :cap] = u[keep]
                s["n_valid"][b, e], s["ecnt"][b, e] = cap, S - cap
        return {name: s[name] for name in out}
    x = (s["x"] if c["kind"] == "route" else s["q"])
    x = x.double().reshape(B, -1)[:, :_d_r(c)] if not c["per_head"] else x.double().reshape(R, D)
    logits = x @ s["W_r"].double()
    if s["bias"] is not None:
        logits = logits + s["bias"].double()
    order = torch.argsort(logits, dim=1, descending=True, stable=True)[:, :k]
    picked = torch.softmax(logits, 1).gather(1, order)
    gates = picked / picked.sum(1, keepdim=True)
    out["topk"], out["gates"] = order.int(), gates
    if c["kind"] == "route":
        return out
    n, u, K, V = s["n_valid"], s["utility"].double(), s["K"], s["V"]
    ecnt = torch.zeros_like(s["ecnt"])
    if not c["per_head"]:
        new = [s["K_new"], s["V_new"]]
        if c["rank"]:
            new = [torch.einsum("bhd,hrd->bhr", s[a].double(), s[w].double()) for a, w in (("K_full", "enc_K"), ("V_full", "enc_V"))]
            out["K_new"], out["V_new"] = new
        victim_of = _victim_values(s)
        for b in range(B):
            for e in order[b].tolist():
                slot = int(n[b, e])
                if slot >= S:
                    v = victim_of(b, e)
                    slot = int((v == v.min()).nonzero()[-1])          # of equal values the higher slot
                    ecnt[b, e] = 1
                else:
                    n[b, e] += 1
                u[b, e, slot] = 0.0
                for t, rows in ((K, new[0]), (V, new[1])):
                    t[b, e, :, slot] = rows[b].to(t.dtype)
                if c["policy"] != "none":
                    s["birth"][b, e, slot] = s["last_access"][b, e, slot] = NOW
                    s["freq"][b, e, slot] = 0
        out["K"], out["V"], out["n_valid"], out["ecnt"] = K, V, n, ecnt
    # query rows by kv head: [B, Hkv, G, D], G = draft queries x heads of the group
    tq, heads = c["tq"], Hq // c["tq"]
    G = Hq // Hkv
    q = s["q"].double().reshape(B, tq, Hkv, heads // Hkv, D).transpose(1, 2).reshape(B, Hkv, G, D)
    y = torch.zeros((B, Hkv, G, D), device=DEV, dtype=torch.float64)
    row_max, row_norm = (torch.zeros((B, Hkv, G), device=DEV, dtype=torch.float64) for _ in range(2))
    scale = 1 / math.sqrt(D)

    def entries(b, e, hk):
        m = int(n[b, e])
        Kd, Vd = K[b, e, hk, :m].double(), V[b, e, hk, :m].double()
        if c["rank"]:
            r = c["rank"]
            Kd, Vd = Kd @ s["U_K"][hk].double(), Vd @ s["U_V"][hk, :r].double()
            if c["value_bias"]:
                Vd = Vd + s["U_V"][hk, r].double()
        return Kd, Vd

    mass = torch.zeros_like(u)
    visited = torch.zeros((B, E), device=DEV, dtype=torch.bool)
    for b in range(B):
        for hk in range(Hkv):
            groups = [(slice(None), b)] if not c["per_head"] else [(slice(g, g + 1), b * Hq + hk * G + g) for g in range(G)]
            for sl, r in groups:
                sel, gt = order[r].tolist(), gates[r]
                parts = []
                for j, e in enumerate(sel):
                    visited[b, e] = True
                    Kd, Vd = entries(b, e, hk)
                    if Kd.shape[0]:
                        parts.append((j, e, (q[b, hk, sl] @ Kd.T) * scale, Vd))
                if not parts:
                    continue
                M = torch.stack([sc.amax(1) for _, _, sc, _ in parts]).amax(0)
                row_max[b, hk, sl] = M
                if c["local"]:
                    norm = sum(gt[j] for j, _, _, _ in parts)
                    ps = [gt[j] / norm * torch.softmax(sc, 1) for j, _, sc, _ in parts]
                    row_norm[b, hk, sl] = norm
                else:
                    ws = [gt[j] * torch.exp(sc - M[:, None]) for j, _, sc, _ in parts]
                    norm = sum(w.sum(1) for w in ws)
                    ps = [w / norm[:, None] for w in ws]
                    row_norm[b, hk, sl] = norm
                for (j, e, sc, Vd), p in zip(parts, ps):
                    y[b, hk, sl] += p @ Vd
                    mass[b, e, :sc.shape[1]] += p.sum(0)
    live = (torch.arange(S, device=DEV) < n[..., None]) & visited[..., None]
    out["utility"] = torch.where(live, c["decay"] * u + mass, u)
    if c["policy"] != "none":
        accessed = live & (mass > 1.0 / S)
        out["birth"], out["last_access"] = s["birth"], torch.where(accessed, NOW, s["last_access"])
        out["freq"] = s["freq"] + accessed.int()

    def caller(t):                       # [B, Hkv, G, ...] -> the tokens' order [B, tq, heads, ...]
        rest = t.shape[3:]
        return t.reshape(B, Hkv, tq, heads // Hkv, *rest).transpose(1, 2).reshape(B, Hq, *rest)

    out["y"], out["row_max"], out["row_norm"] = caller(y), caller(row_max), caller(row_norm)
    if c["feedback"]:
        load = s["load"] + torch.bincount(order.flatten(), minlength=E).int()
        out["load"], out["bias"] = load, -PENALTY * (load.double() - load.double().mean())
    return out


def _victim_values(s):
    """(b, e) -> the values an eviction from the full shard minimises."""
    c = s["case"]
    if c["policy"] == "none":
        return lambda b, e: s["utility"][b, e]
    if c["policy"] == "sl":
        return lambda b, e: (NOW - s["birth"][b, e] < NOW * 3 // 4).double()
    if c["policy"] == "lru":
        return lambda b, e: -(NOW - s["last_access"][b, e]).double()
    return lambda b, e: 0.5 * s["freq"][b, e].double() - (NOW - s["last_access"][b, e]).double()
