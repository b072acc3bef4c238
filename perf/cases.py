"""The calls this framework is timed on: whole layers, the expert products, the router, the predictor and the
row movement, each through the entry points a program calls, from a decode step of a few dozen tokens to a
batch of 65536.

A case is a dict of plain values:

  kind "layer"    MoeLayer.forward (MoeLayerTopK.forward when k > 1): router -> replica plan + dispatch -> expert FFN
                  -> combine.  Tokens carry the direction of the expert they belong to, as after training, so the
                  routing decision is clear and does not hang on the order of a sum.
  kind "ffn"      moe_expert_ffn on the tables of one batch, rows gathered through the permutation
  kind "route"    moe_route / moe_route_topk with a popularity bias on random logits
  kind "predict"  sru_predict (SRU stack, optional sparsemax attention, head) with its logits
  kind "move"     moe_dispatch with the row copy, then moe_combine: a program whose experts run elsewhere

Popularity of the experts: Zipf(zipf), or a share `hot` of the tokens on one expert and Zipf over the rest.
Slot capacity: cf * k * T / E rounded up, at least 4.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2605_11537_amd as moe

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f32": 4}


# ------------------------------------------------------------------------------------------------- the cases
def _layer(dtype, T, d, F, E, R, zipf=1.0, hot=0.0, cf=1.25, k=1, residual=0, renorm=False):
    return dict(kind="layer", dtype=dtype, T=T, d=d, F=F, E=E, R=R, zipf=zipf, hot=hot, cf=cf, k=k,
                residual=residual, renorm=renorm)


def listed():
    return [
        # a toy-sized binary32 layer: everything is cache resident, launches and latency are all there is
        dict(name="layer_f32_tiny", **_layer("f32", 512, 64, 256, 8, 4, zipf=1.2)),
        # binary32 inference of a small model at an odd batch
        dict(name="layer_f32_1500", **_layer("f32", 1500, 512, 2048, 32, 8)),
        # one decode step: a few dozen sequences, one token each
        dict(name="layer_decode_37", **_layer("bf16", 37, 768, 3072, 128, 16)),
        # the usual evaluation batch of a 128-expert layer (8 sequences of 512 tokens)
        dict(name="layer_4096", **_layer("bf16", 4096, 768, 3072, 128, 16)),
        # the same batch under top-3 routing
        dict(name="layer_top3_4096", **_layer("bf16", 4096, 768, 3072, 128, 16, k=3)),
        # a large batch with half of its tokens on one expert, inside a residual stack
        dict(name="layer_skew_65536", **_layer("bf16", 65536, 768, 3072, 256, 64, hot=0.5, cf=4.0, residual=1)),
        # the expert products of a 256-expert layer at capacity factor 1
        dict(name="ffn_16384", kind="ffn", dtype="bf16", T=16384, d=768, F=3072, E=256, R=32, zipf=1.1, hot=0.0, cf=1.0),
        # the gate of a 64-expert layer on a ragged batch
        dict(name="route_e64_3001", kind="route", dtype="bf16", T=3001, d=768, E=64, k=1, renorm=False, zipf=1.0),
        # the gate of a 256-expert layer on a prefill batch
        dict(name="route_e256_16384", kind="route", dtype="bf16", T=16384, d=768, E=256, k=1, renorm=False, zipf=1.1),
        # the predictor on a few long sequences of odd length
        dict(name="predict_2x777", kind="predict", B=5, L=777, n_in=768, n_h=256, layers=2, n_out=128, attention=False),
        # the ten-layer predictor with sparse attention on the usual evaluation batch
        dict(name="predict_10_attention", kind="predict", B=8, L=512, n_in=768, n_h=256, layers=10, n_out=128,
             attention=True),
        # rows out to the experts and back at the large batch
        dict(name="move_65536", kind="move", dtype="bf16", T=65536, d=768, E=256, R=64, zipf=1.0, hot=0.5, cf=4.0,
             residual=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["layer", "ffn", "route", "predict", "move"], [7, 3, 4, 3, 3])[0]
    if kind == "predict":
        L = _log_int(rng, 16, 1024)
        n_out = rng.choice([64, 128, 128, 256])
        return dict(kind=kind, B=rng.randint(1, min(16, max(1, 8192 // L))), L=L, n_in=rng.choice([128, 256, 512, 768]),
                    n_h=rng.choice([128, 256]), layers=rng.randint(1, 10), n_out=n_out, attention=rng.random() < 0.5)
    zipf = round(rng.uniform(0.6, 1.4), 2)
    if kind == "route":
        E = rng.choice([8, 16, 24, 32, 64, 100, 128, 128, 256, 256])
        dtype = "bf16" if rng.random() < 0.75 else "f32"
        top = 65536 if dtype == "bf16" and E >= 128 else 8192
        return dict(kind=kind, dtype=dtype, T=_log_int(rng, 16, top), d=rng.choice([128, 256, 384, 512, 768, 1024]), E=E,
                    k=rng.choice([1, 1, 1, 2, 3]), renorm=rng.random() < 0.5, zipf=zipf)
    dtype = "bf16" if rng.random() < 0.8 else "f32"
    hot = rng.choice([0.0, 0.0, 0.0, round(rng.uniform(0.1, 0.6), 2)])
    cf = rng.choice([1.0, 1.25, 2.0, 4.0])
    if kind == "move":
        E = rng.choice([8, 32, 64, 128, 256])
        return dict(kind=kind, dtype=dtype, T=_log_int(rng, 16, 65536 if dtype == "bf16" else 32768),
                    d=rng.choice([256, 384, 512, 768]), E=E, R=E // 8 * rng.randint(0, 2), zipf=zipf, hot=hot, cf=cf,
                    residual=rng.randint(0, 1))
    if dtype == "f32":
        d, F = rng.choice([(64, 256), (256, 1024), (512, 2048)])
        T, E = _log_int(rng, 16, 2048), rng.choice([8, 16, 32, 64])
    else:
        d, F = rng.choice([(256, 1024), (384, 1536), (512, 2048), (768, 3072), (768, 3072), (1024, 4096)])
        E = rng.choice([8, 16, 32, 64, 128, 128, 256]) if d < 1024 else rng.choice([8, 16, 32, 64, 128])
        T = _log_int(rng, 16, 65536 if E == 256 and d <= 768 else 16384)
    R = E // 8 * rng.randint(0, 2)
    if kind == "ffn":
        return dict(kind=kind, dtype=dtype, T=T, d=d, F=F, E=E, R=R, zipf=zipf, hot=hot, cf=cf)
    k = rng.choice([1, 1, 1, 2, 3]) if T <= 16384 else 1
    return _layer(dtype, T, d, F, E, R, zipf=zipf, hot=hot, cf=cf, k=k, residual=rng.randint(0, 1),
                  renorm=rng.random() < 0.5)


# ------------------------------------------------------------------------------------------------- inputs
def _popularity(c):
    """Share of the tokens each popularity rank gets (rank 0 is the hottest)."""
    E, hot = c["E"], c.get("hot", 0.0)
    if hot <= 0.0:
        w = np.arange(1, E + 1, dtype=np.float64) ** -c["zipf"]
        return w / w.sum()
    w = np.arange(1, E, dtype=np.float64) ** -c["zipf"]
    return np.concatenate([[hot], (1.0 - hot) * w / w.sum()])


def _capacity(c):
    return max(4, math.ceil(c["cf"] * c.get("k", 1) * c["T"] / c["E"]))


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype).mul_(std)


def _shares(c, g):
    """Popularity of every expert id: the ranks are dealt to the ids at random."""
    order = torch.randperm(c["E"], generator=g, device="cuda")
    return torch.from_numpy(_popularity(c)).cuda()[order]


def _ids(c, g):
    """[k, T] expert ids, distinct within a token."""
    p, T, k = _shares(c, g), c["T"], c.get("k", 1)
    if k == 1:
        return torch.multinomial(p, T, replacement=True, generator=g).view(1, T)
    return torch.multinomial(p.expand(T, -1), k, replacement=False, generator=g).t().contiguous()


def _expert_weights(c, g):
    dt = DTYPES[c["dtype"]]
    return _normal(g, (c["E"], c["d"], c["F"]), 0.02, dt), _normal(g, (c["E"], c["F"], c["d"]), 0.02, dt)


def _layer_inputs(c, seed):
    g, dt = _generator(seed), DTYPES[c["dtype"]]
    T, d, E = c["T"], c["d"], c["E"]
    z = _ids(c, g)
    u = torch.randn((E, d), generator=g, device="cuda")
    u /= u.norm(dim=1, keepdim=True)
    x = torch.randn((T, d), generator=g, device="cuda")
    for j in range(z.shape[0]):
        x += (8.0 + 1.5 * (z.shape[0] - 1 - j)) * u[z[j]]
    w_router = 0.02 * torch.randn((d, E), generator=g, device="cuda") + u.t()
    b_router = 0.02 * torch.randn(E, generator=g, device="cuda")
    w1, w2 = _expert_weights(c, g)
    return dict(x=x.to(dt), w_router=w_router.to(dt).contiguous(), b_router=b_router, w1=w1, w2=w2)


def _ffn_inputs(c, seed):
    g = _generator(seed)
    ids = _ids(c, g).view(-1).to(torch.int32)
    x = _normal(g, (c["T"], c["d"]), 1.0, DTYPES[c["dtype"]])
    w1, w2 = _expert_weights(c, g)
    return dict(x=x, ids=ids, w1=w1, w2=w2)


def _route_inputs(c, seed):
    g, dt = _generator(seed), DTYPES[c["dtype"]]
    p = _shares(c, g)
    spread = 0.02 * math.sqrt(c["d"])                 # standard deviation of one logit
    bias = (0.5 * spread * torch.log(p / p.max())).float()
    return dict(x=_normal(g, (c["T"], c["d"]), 1.0, dt), w_router=_normal(g, (c["d"], c["E"]), 0.02, dt), b_router=bias)


def _predict_inputs(c, seed):
    g, bf = _generator(seed), torch.bfloat16
    n_h = c["n_h"]
    out = dict(emb=_normal(g, (c["B"], c["L"], c["n_in"]), 1.0, bf), w_cat=[], b_f=[], b_r=[])
    n = c["n_in"]
    for _ in range(c["layers"]):
        out["w_cat"].append(_normal(g, (n, (3 if n == n_h else 4) * n_h), 0.05, bf))
        out["b_f"].append(_normal(g, (n_h,), 0.1, torch.float32))
        out["b_r"].append(_normal(g, (n_h,), 0.1, torch.float32))
        n = n_h
    out["w_head"] = _normal(g, (n_h, c["n_out"]), 0.05, bf)
    out["b_head"] = _normal(g, (c["n_out"],), 0.1, torch.float32)
    return out


def _move_inputs(c, seed):
    g, dt = _generator(seed), DTYPES[c["dtype"]]
    T, d = c["T"], c["d"]
    ids = _ids(c, g).view(-1).to(torch.int32)
    return dict(ids=ids, x=_normal(g, (T, d), 1.0, dt), y=_normal(g, (T, d), 0.5, dt),
                prob=torch.rand(T, generator=g, device="cuda") * 0.8 + 0.2)


def _packed(w):
    return moe.moe_pack_weights(w) if w.dtype == torch.bfloat16 else w


def _router_image(w, d, E):
    """Static router weights are packed once wherever the library takes the packed image."""
    if w.dtype == torch.bfloat16 and E in (128, 256) and d % 128 == 0:
        return moe.moe_pack_weights(w[None].contiguous())[0], moe.LAYOUT_PACKED
    return w, moe.LAYOUT_PLAIN


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    c = case
    if c["kind"] == "predict":
        i = _predict_inputs(c, seed)
        w = moe.SruWeights(i["w_cat"], i["b_f"], i["b_r"], i["w_head"], i["b_head"], pack=c["n_out"] in (128, 256),
                           attention=c["attention"])
        need = moe.lib().sru_predict_workspace_bytes(ctypes.byref(w.c), c["B"], c["L"], moe.MOE_BF16)
        return dict(case=c, emb=i["emb"], w=w, ws=_workspace(need),
                    pred=torch.zeros(c["B"] * c["L"], dtype=torch.int32, device="cuda"))
    dt, T, d, E = DTYPES[c["dtype"]], c["T"], c["d"], c["E"]
    if c["kind"] == "route":
        i = _route_inputs(c, seed)
        wr, layout = _router_image(i["w_router"], d, E)
        k = c["k"]
        idx = torch.zeros((k, T) if k > 1 else T, dtype=torch.int32, device="cuda")
        need = moe.lib().moe_route_workspace_bytes(T, d, E, moe.MOE_BF16 if c["dtype"] == "bf16" else moe.MOE_F32)
        return dict(case=c, x=i["x"], wr=wr, layout=layout, b=i["b_router"], ws=_workspace(need),
                    out=(idx, torch.zeros(idx.shape, dtype=torch.float32, device="cuda")))
    C = _capacity(c)
    if c["kind"] == "layer":
        i = _layer_inputs(c, seed)
        wr, layout = _router_image(i["w_router"], d, E)
        if c["k"] == 1:
            layer = moe.MoeLayer(T, d, c["F"], E, c["R"], C, dt)
        else:
            layer = moe.MoeLayerTopK(T, d, c["F"], E, c["k"], c["R"], C, dt, renormalize=c["renorm"])
        return dict(case=c, layer=layer, x=i["x"], wr=wr, layout=layout, b=i["b_router"], w1=_packed(i.pop("w1")),
                    w2=_packed(i.pop("w2")))
    if c["kind"] == "ffn":
        i = _ffn_inputs(c, seed)
        plan, disp = moe.moe_plan_dispatch(i["ids"], i["ids"], E, c["R"], C)
        code = moe.MOE_BF16 if c["dtype"] == "bf16" else moe.MOE_F32
        need = moe.lib().moe_expert_ffn_workspace_bytes(T, E + c["R"], d, c["F"], code)
        return dict(case=c, x=i["x"], w1=_packed(i.pop("w1")), w2=_packed(i.pop("w2")), plan=plan, disp=disp,
                    y=torch.zeros(T, d, dtype=dt, device="cuda"), ws=_workspace(need))
    i = _move_inputs(c, seed)
    plan = moe.replica_plan(i["ids"], E, c["R"], C)
    n = E + c["R"]
    i32 = lambda m: torch.zeros(m, dtype=torch.int32, device="cuda")  # noqa: E731
    disp = dict(counts=i32(E), kept=i32(E), expert_offset=i32(E + 1), slot_offset=i32(n + 1), perm=i32(T), inv=i32(T),
                x_perm=torch.zeros(T, d, dtype=dt, device="cuda"))
    return dict(case=c, C=C, x=i["x"], y=i["y"], prob=i["prob"], ids=i["ids"], plan=plan, disp=disp,
                ws=_workspace(moe.lib().moe_dispatch_workspace_bytes(T, E)), out=torch.zeros(T, d, dtype=dt, device="cuda"))


# ------------------------------------------------------------------------------------------------- one pass
def run(state):
    s, c = state, state["case"]
    if c["kind"] == "predict":
        pred, logits = moe.sru_predict(s["emb"], s["w"], want_logits=True, out=s["pred"], ws=s["ws"])
        return dict(pred=pred, logits=logits)
    if c["kind"] == "route":
        if c["k"] == 1:
            idx, prob, _ = moe.moe_route(s["x"], s["wr"], s["b"], out=s["out"], ws=s["ws"], w_layout=s["layout"])
        else:
            idx, prob, _ = moe.moe_route_topk(s["x"], s["wr"], s["b"], c["k"], c["renorm"], out=s["out"], ws=s["ws"],
                                              w_layout=s["layout"])
        return dict(idx=idx, prob=prob)
    if c["kind"] == "layer":
        layer = s["layer"]
        out = layer.forward(s["x"], s["wr"], s["b"], s["w1"], s["w2"], residual=c["residual"], router_layout=s["layout"])
        return dict(out=out, idx=layer.route_out[0], prob=layer.route_out[1], replicas=layer.plan_out["replicas"],
                    inv=layer.disp_out["inv"])
    if c["kind"] == "ffn":
        disp, plan = s["disp"], s["plan"]
        return moe.moe_expert_ffn(s["x"], s["w1"], s["w2"], disp["slot_offset"], plan["slot_expert"], plan["n_slots"],
                                  c["E"], c["F"], out=s["y"], ws=s["ws"], row_index=disp["perm"])
    disp = moe.moe_dispatch(s["x"], s["ids"], s["plan"]["replicas"], c["E"], s["C"], c["E"] + c["R"], out=s["disp"],
                            ws=s["ws"])
    out = moe.moe_combine(s["y"], s["x"], disp["inv"], s["prob"], c["residual"], out=s["out"])
    return dict(out=out, **disp)


# ------------------------------------------------------------------------------------------------- cost
def _plan(counts, E, R, C):
    """Replicas per expert: as many slots of C tokens as it needs; over budget, in proportion to the slots still
    wanted, rounded down, the rest one by one to the fullest slot (lowest id first)."""
    n = [int(v) for v in counts]
    want = [max(0, -(-v // C) - 1) for v in n]
    D = sum(want)
    if D <= R:
        return [1 + w for w in want]
    r = [1 + R * w // D for w in want]
    for _ in range(R - sum(r) + E):
        best = -1
        for e in range(E):
            if r[e] < 1 + want[e] and (best < 0 or n[e] * r[best] > n[best] * r[e]):
                best = e
        if best < 0:
            break
        r[best] += 1
    return r


def _expected(c):
    """(assignments kept, experts with a token) to expect of this case."""
    p, n, C = _popularity(c), c["T"] * c.get("k", 1), _capacity(c)
    counts = p * n
    r = _plan(np.round(counts), c["E"], c["R"], C)
    kept = float(sum(min(a, b * C) for a, b in zip(counts, r)))
    return kept, float(np.sum(1.0 - (1.0 - np.minimum(p, 1.0)) ** n))


def work(case):
    c = case
    if c["kind"] == "predict":
        T, n, by, fl = c["B"] * c["L"], c["n_in"], 0, 0
        by += T * n * 2 + T * 4 + T * c["n_out"] * 4 + c["n_h"] * c["n_out"] * 2
        fl += 2 * T * c["n_h"] * c["n_out"]
        for _ in range(c["layers"]):
            cols = (3 if n == c["n_h"] else 4) * c["n_h"]
            by += n * cols * 2
            fl += 2 * T * n * cols
            n = c["n_h"]
        if c["attention"]:
            fl += 4 * T * c["L"] * c["n_h"]
        return {"bytes": by, "flops": fl}
    b, T, d, E = SIZE[c["dtype"]], c["T"], c["d"], c["E"]
    gate = {"bytes": T * d * b + d * E * b + 8 * T * c.get("k", 1), "flops": 2 * T * d * E}
    if c["kind"] == "route":
        return gate
    kept, active = _expected(c)
    if c["kind"] == "move":
        dropped = T if c["residual"] else T - kept
        return {"bytes": 2 * kept * d * b + kept * d * b + dropped * d * b + T * d * b + 12 * T, "flops": 2 * kept * d}
    weights = active * 2 * d * c["F"] * b
    flops = 4 * kept * d * c["F"]
    if c["kind"] == "ffn":
        return {"bytes": weights + 2 * kept * d * b + 4 * T, "flops": flops}
    return {"bytes": weights + gate["bytes"] + T * d * b, "flops": flops + gate["flops"] + 2 * kept * d}


def tolerance(case):
    """About four times what each path differs by from exact() where it is all rounding."""
    c = case
    if c["kind"] == "predict":      # bf16 states handed from layer to layer; ids may differ where two logits are close
        return {"rel": 1e-2, "max": 0.2, "differ": 0.01}
    if c["kind"] == "route":        # binary32 sums of up to 1024 products; ids may differ where two logits tie
        return {"rel": 4e-6, "max": 1e-4, "differ": 1e-3}
    if c["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4, "differ": 1e-4}
    return {"rel": 1e-2, "max": 0.1, "differ": 1e-4}


# ------------------------------------------------------------------------------------------------- 64-bit results
def _rank(ids, E):
    """Rank of every entry among the earlier entries with the same id."""
    order = torch.sort(ids, stable=True)[1]
    counts = torch.bincount(ids, minlength=E)
    start = torch.cumsum(counts, 0) - counts
    rank = torch.empty_like(ids)
    rank[order] = torch.arange(ids.numel(), device=ids.device) - start[ids[order]]
    return rank, counts


def _tables(c, ids):
    """(kept mask of every entry, its row among the kept ones) for int64 ids in dispatch order."""
    rank, counts = _rank(ids, c["E"])
    r = torch.tensor(_plan(counts.tolist(), c["E"], c["R"], _capacity(c)), device=ids.device)
    kept = torch.minimum(counts, r * _capacity(c))
    first = torch.cumsum(kept, 0) - kept
    keep = rank < kept[ids]
    return keep, first[ids] + rank


def _ffn64(x, ids, w1, w2):
    """relu(x W1[e]) W2[e] for rows x with expert ids."""
    y = torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    for e in torch.unique(ids).tolist():
        rows = (ids == e).nonzero().view(-1)
        y[rows] = torch.relu(x[rows].double() @ w1[e].double()) @ w2[e].double()
    return y


def _gate64(c, i):
    logits = i["x"].double() @ i["w_router"].double() + i["b_router"].double()
    p = torch.softmax(logits, 1)
    idx = torch.sort(logits, dim=1, descending=True, stable=True)[1][:, : c["k"]]
    w = torch.gather(p, 1, idx)
    if c["k"] > 1 and c["renorm"]:
        w = w / w.sum(1, keepdim=True)
    return idx.t().contiguous(), w.t().contiguous()


def _sru64(c, i):
    h = i["emb"].double()
    B, L, n_h = c["B"], c["L"], c["n_h"]
    for w, b_f, b_r in zip(i["w_cat"], i["b_f"], i["b_r"]):
        u = (h.reshape(B * L, -1) @ w.double()).view(B, L, -1)
        f, r = torch.sigmoid(u[..., n_h:2 * n_h] + b_f.double()), torch.sigmoid(u[..., 2 * n_h:3 * n_h] + b_r.double())
        v = (1 - f) * u[..., :n_h]
        s, state = torch.empty_like(v), torch.zeros_like(v[:, 0])
        for t in range(L):
            state = torch.addcmul(v[:, t], f[:, t], state)
            s[:, t] = state
        h = r * torch.tanh(s) + (1 - r) * (u[..., 3 * n_h:] if u.shape[2] == 4 * n_h else h)
    if c["attention"]:
        out = torch.empty_like(h)
        for b in range(B):
            s = h[b] @ h[b].t() / math.sqrt(n_h)
            v = torch.sort(s, dim=1, descending=True)[0]
            cum = torch.cumsum(v, 1)
            m = torch.arange(1, L + 1, device=s.device, dtype=torch.float64)
            size = (1 + m * v > cum).sum(1, keepdim=True)
            tau = (torch.gather(cum, 1, size - 1) - 1) / size
            out[b] = h[b] + torch.clamp(s - tau, min=0) @ h[b]
        h = out
    return h.reshape(B * L, n_h) @ i["w_head"].double() + i["b_head"].double()


def exact(case, seed):
    c = case
    if c["kind"] == "predict":
        return dict(pred=None, logits=_sru64(c, _predict_inputs(c, seed)))
    if c["kind"] == "route":
        _, w = _gate64(c, _route_inputs(c, seed))
        return dict(idx=None, prob=w if c["k"] > 1 else w.view(-1))
    T, d, k = c["T"], c["d"], c.get("k", 1)
    if c["kind"] == "ffn":
        i = _ffn_inputs(c, seed)
        ids = i["ids"].long()
        keep, row = _tables(c, ids)
        y = torch.zeros((T, d), dtype=torch.float64, device="cuda")
        y[row[keep]] = _ffn64(i["x"][keep], ids[keep], i["w1"], i["w2"])
        return y
    if c["kind"] == "move":
        i = _move_inputs(c, seed)
        x = i["x"].double()
        keep, row = _tables(c, i["ids"].long())
        x_perm = torch.zeros_like(x)
        x_perm[row[keep]] = x[keep]
        out = x.clone()
        out[keep] = (x[keep] if c["residual"] else 0.0) + i["prob"][keep, None].double() * i["y"].double()[row[keep]]
        return dict(out=out, counts=None, kept=None, expert_offset=None, slot_offset=None, perm=None, inv=None, x_perm=x_perm)
    i = _layer_inputs(c, seed)
    idx, w = _gate64(c, i)
    ids, flat = idx.reshape(-1), w.reshape(-1)
    keep, _ = _tables(c, ids)
    entries = keep.nonzero().view(-1)
    y = _ffn64(i["x"][entries % T], ids[entries], i["w1"], i["w2"]) * flat[entries, None]
    x = i["x"].double()
    out = (x if c["residual"] else torch.zeros_like(x)).index_add(0, entries % T, y)
    none = torch.ones(T, dtype=torch.bool, device="cuda")
    none[entries % T] = False
    out[none] = x[none]
    return dict(out=out, idx=None, prob=w if k > 1 else w.view(-1), replicas=None, inv=None)
