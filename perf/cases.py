"""The workloads that performance work on this package is measured on.

Each case is one piece of what a program does with the package, called through
`paper_2604_21290_amd.api`: a graph build, an update, a ViG layer, a full block,
a whole stack.  Shapes are the ViG-Ti, ViG-B and ViG-Pyramid stages of
`paper_2604_21290_amd.inputs` and generic odd ones around them.

listed()          the fixed cases
draw(rng)         one more case of the same ranges
prepare(case, s)  inputs, weights, outputs, workspaces and handles of a case
run(state)        one pass; returns the outputs
work(case)        bytes and operations one pass cannot do without
exact(case, s)    the same outputs in float64, from the definitions
tolerance(case)   what two correct implementations may differ by
"""
from __future__ import annotations

import math

import torch

from paper_2604_21290_amd import api

PARAMS = api.VIG_PARAMS
FUSED, LOOKAHEAD, STANDARD = "fused", "lookahead", "standard"
SCHEDULE = {FUSED: api.GL_SCHED_LOOKAHEAD_FUSED, LOOKAHEAD: api.GL_SCHED_LOOKAHEAD,
            STANDARD: api.GL_SCHED_STANDARD}


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def _case(kind, B, H, W, C, k=9, d=1, dtype="bf16", pool=1, L=1, ramp=4, schedule=FUSED,
          Cout=0, heads=0, features="unit", bias=True):
    """kind        what is called (see `run`)
    B, H, W, C     images, node grid, channels
    k, d           neighbours per node, dilation (of a stack's first block)
    pool           keys are pooled pool x pool
    L, ramp        blocks of a stack; the dilation grows by one every `ramp` blocks
    Cout, heads    output channels (0: C) and heads (0: dense) of an update
    features       "unit": normalised noise; "mixture": regions of alike nodes"""
    return dict(kind=kind, B=B, H=H, W=W, C=C, k=k, d=d, dtype=dtype, pool=pool, L=L, ramp=ramp,
                schedule=schedule, Cout=Cout or C, heads=heads, features=features, bias=bias)


def listed():
    return [
        # one image, one layer in fp32: the smallest call, all launch and latency
        dict(_case("layer", 1, 14, 14, 192, dtype="fp32", bias=False), name="layer_single_fp32"),
        # an odd grid and width in fp32, a wider dilated neighbourhood
        dict(_case("layer", 3, 27, 19, 204, k=12, d=3, dtype="fp32"), name="layer_ragged_fp32"),
        # the benchmark's stack: ViG-Ti, 12 graph + update blocks on a batch of 32
        dict(_case("stack", 32, 14, 14, 192, L=12, bias=False), name="stack_vig_ti"),
        # the first pyramid stage's two blocks: many nodes, narrow, pooled keys
        dict(_case("stack", 32, 56, 56, 80, pool=4, L=2, schedule=LOOKAHEAD, bias=False),
             name="stack_pyr_s1"),
        # the graph of a high-resolution grid: every node against every node
        dict(_case("knn", 8, 56, 56, 96, k=16, d=2, features="mixture"), name="knn_hires"),
        # the graph of ViG-Ti at 448 x 448 (784 nodes) in its later, dilated blocks
        dict(_case("knn", 32, 28, 28, 192, d=3), name="knn_vig_ti_448"),
        # the update of ViG-B, whose weights are wide
        dict(_case("mrconv", 64, 14, 14, 640), name="mrconv_vig_b"),
        # the multi-head update of ViG-Ti
        dict(_case("mrconv", 32, 14, 14, 192, heads=16), name="mrconv_heads_vig_ti"),
        # from the first pyramid stage to the second: max pooling, then the projection
        dict(_case("stage", 32, 56, 56, 80, pool=2, Cout=160), name="stage_pyr_s1_s2"),
        # one full ViG-B block and the graph of the next: the matrix products
        dict(_case("vig_block", 64, 14, 14, 640, d=2), name="vig_block_b"),
        # a whole ViG-Ti of full blocks: a batch, and one image being served
        dict(_case("vig_stack", 32, 14, 14, 192, L=12), name="vig_stack_ti"),
        dict(_case("vig_stack", 1, 14, 14, 192, L=12), name="vig_stack_ti_b1"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost_us(c):
    """A rough time of a case, to keep the drawn ones within the listed ones."""
    w = work(c)
    B, N, M, C = c["B"], _nodes(c), _keys(c), c["C"]
    builds = {"knn": 1, "layer": 1, "vig_block": 1, "stack": c["L"], "vig_stack": c["L"]}.get(c["kind"], 0)
    rate = 250e6 if c["dtype"] == "bf16" else 25e6
    return w["flops"] / rate + w["bytes"] / 2e6 + builds * B * N * M / 5e5


def draw(rng):
    while True:
        kind = rng.choice(["layer", "stack", "knn", "mrconv", "stage", "vig_block", "vig_stack"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        B = _log_int(rng, 1, 64)
        pool = rng.choice([1, 1, 2, 4]) if kind != "stage" else 2
        H = pool * _log_int(rng, max(2, 7 // pool), 56 // pool)
        W = pool * _log_int(rng, max(2, 7 // pool), 56 // pool)
        C = _log_int(rng, 6, 80) * 8 + (0 if dtype == "bf16" else rng.choice([0, 4]))
        k = rng.choice([4, 7, 9, 9, 9, 12, 16])
        d = rng.randint(1, 4)
        # a two-block lookahead stack builds both graphs from its input, so its
        # outputs do not hang on how an earlier block was rounded
        c = _case(kind, B, H, W, C, k=k, d=d, dtype=dtype, pool=pool,
                  L=2 if kind in ("stack", "vig_stack") else 1, ramp=rng.choice([1, 4]),
                  schedule=rng.choice([FUSED, LOOKAHEAD]), features=rng.choice(["unit", "mixture"]),
                  Cout=_log_int(rng, 6, 80) * 8 if kind in ("mrconv", "stage") else C,
                  bias=rng.random() < 0.5)
        if kind == "mrconv" and rng.random() < 0.25:
            c["heads"], c["Cout"] = rng.choice([h for h in (2, 4, 8, 16) if C % (4 * h) == 0] or [1]), C
        if k * max(_dilations(c)) > min(_keys(c), api.GL_MAX_KD) or _cost_us(c) > 500:
            continue
        return c


# ---------------------------------------------------------------------------
# geometry
# ---------------------------------------------------------------------------
def _nodes(c):
    return c["H"] * c["W"]


def _keys(c):
    return (c["H"] // c["pool"]) * (c["W"] // c["pool"])


def _dilations(c):
    return [c["d"] + l // c["ramp"] for l in range(c["L"])]


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _graph_d(c):
    """The dilation of the graph a single call is handed (a block builds the
    next one with the case's own)."""
    return c["d"]


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _features(c, g):
    B, H, W, C = c["B"], c["H"], c["W"], c["C"]
    x = torch.randn((B, H * W, C), generator=g, device="cuda")
    if c["features"] == "mixture":
        # eight regions of the grid (nearest of eight sites), each around a mean
        mu = torch.randn((B, 8, C), generator=g, device="cuda")
        site = torch.rand((B, 8, 2), generator=g, device="cuda") * torch.tensor([H, W], device="cuda")
        yy, xx = torch.meshgrid(torch.arange(H, device="cuda"), torch.arange(W, device="cuda"),
                                indexing="ij")
        pos = torch.stack([yy.reshape(-1), xx.reshape(-1)], 1).float()
        comp = ((pos[None, :, None, :] - site[:, None, :, :]) ** 2).sum(-1).argmin(-1)
        x = torch.gather(mu, 1, comp[:, :, None].expand(-1, -1, C)) + 0.5 * x
    else:
        x = x / x.norm(dim=-1, keepdim=True)
    return x.to(_dtype(c)).contiguous()


def _uniform(g, shape, bound, dt):
    return ((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * bound).to(dt)


def _weight(c, g, out, fan_in, scale=1.0):
    return _uniform(g, (out, fan_in), scale * math.sqrt(6.0 / fan_in), _dtype(c))


def _bias(c, g, n):
    return _uniform(g, (n,), 0.1, _dtype(c)) if c["bias"] else None


def _vig_weights(c, g):
    """One full block's weights; the layers that end a residual branch are small,
    as a stack without normalisation layers needs them."""
    C = c["C"]
    p = {"W_in": _weight(c, g, C, C), "W_upd": _weight(c, g, C, 2 * C),
         "W_out": _weight(c, g, C, C, 0.2), "W_1": _weight(c, g, 4 * C, C),
         "W_2": _weight(c, g, C, 4 * C, 0.2)}
    for name, n in (("b_in", C), ("b_upd", C), ("b_out", C), ("b_1", 4 * C), ("b_2", C)):
        p[name] = _bias(c, g, n)
    return p


def _pooled(x, c, how):
    B, N, C = x.shape
    r = c["pool"]
    v = x.reshape(B, c["H"] // r, r, c["W"] // r, r, C)
    v = v.mean(dim=(2, 4)) if how == "mean" else v.amax(dim=(2, 4))
    return v.reshape(B, -1, C)


def _neighbours(x, keys, k, d):
    """Dilated k nearest keys of each row by the distance of the normalised
    rows, nearest first, ties to the lower index."""
    out = []
    for b in range(x.shape[0]):
        q = x[b] / x[b].norm(dim=-1, keepdim=True).clamp_min(1e-12)
        s = keys[b] / keys[b].norm(dim=-1, keepdim=True).clamp_min(1e-12)
        dist = (q * q).sum(-1, keepdim=True) + (s * s).sum(-1) - 2 * (q @ s.t().contiguous())
        out.append(dist.sort(dim=-1, stable=True).indices[:, :k * d:d])
    return torch.stack(out)


def _data(c, seed):
    """The inputs of a case, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    kind, C, Co = c["kind"], c["C"], c["Cout"]
    x = _features(c, g)
    s = {"x": x}
    if kind in ("layer", "mrconv", "vig_block"):
        # a block is handed the graph of the features before its own: of alike
        # features here, of which FC1 keeps the neighbourhoods
        f = _pooled(x.float(), c, "mean") if c["pool"] > 1 else x.float()
        if kind != "layer":
            s["idx"] = _neighbours(x.float(), f, c["k"], _graph_d(c)).int().contiguous()
        if kind == "mrconv" and c["pool"] > 1:
            s["keys"] = f.to(x.dtype).contiguous()
    if kind in ("layer", "mrconv"):
        h = c["heads"]
        s["W"] = (_weight(c, g, C, 2 * C // h).reshape(h, C // h, 2 * C // h).contiguous() if h
                  else _weight(c, g, Co, 2 * C))
        s["b"] = _bias(c, g, Co)
    elif kind == "stage":
        s["W"], s["b"] = _weight(c, g, Co, C), _bias(c, g, Co)
    elif kind == "stack":
        s["W"] = torch.stack([_weight(c, g, C, 2 * C) for _ in range(c["L"])])
        s["b"] = torch.stack([_bias(c, g, C) for _ in range(c["L"])]) if c["bias"] else None
    elif kind in ("vig_block", "vig_stack"):
        s["p"] = [_vig_weights(c, g) for _ in range(c["L"])]
    return s


def prepare(case, seed):
    c, s = case, _data(case, seed)
    x, kind = s["x"], c["kind"]
    B, N, C = x.shape
    s["case"] = c
    new = lambda *shape: torch.empty(shape, dtype=x.dtype, device="cuda")  # noqa: E731
    idx = lambda: torch.empty((B, N, c["k"]), dtype=torch.int32, device="cuda")  # noqa: E731
    if kind in ("layer", "knn"):
        s["graph"] = idx()
        s["pooled"] = new(B, _keys(c), C) if c["pool"] > 1 else None
    if kind in ("layer", "mrconv"):
        s["out"] = new(B, N, c["Cout"])
        s["ws"] = (api.mrconv_heads_workspace(B, N, C, c["k"], c["heads"], x.dtype, x.device)
                   if c["heads"] else api.mrconv_workspace(B, N, C, c["k"], c["Cout"], x.dtype, x.device))
    if kind == "stage":
        s["pooled"], s["out"] = new(B, _keys(c), C), new(B, _keys(c), c["Cout"])
    if kind in ("stack", "vig_block", "vig_stack"):
        s["la"] = api.Lookahead(torch.cuda.current_stream(), torch.cuda.Stream())
        s["out"] = new(B, N, C)
        s["ws"] = (api.make_stack_workspace(x, c["H"], c["W"], c["k"], c["pool"]) if kind == "stack"
                   else api.vig_workspace(x, c["k"], c["H"], c["W"], c["pool"]))
    if kind == "vig_block":
        s["u"], s["graph"] = new(B, N, C), idx()
    return s


def run(s):
    c, x = s["case"], s["x"]
    kind, H, W, k, d, r = c["kind"], c["H"], c["W"], c["k"], c["d"], c["pool"]
    if kind in ("layer", "knn"):
        # a graph build, and in a layer the update on that graph
        keys = api.pool_keys(x, H, W, r, out=s["pooled"]) if r > 1 else None
        api.knn_graph(x, k, d, keys=keys, out=s["graph"])
        if kind == "knn":
            return {"idx": s["graph"]}
        api.mrconv(x, s["graph"], s["W"], s["b"], keys=keys, out=s["out"], ws=s["ws"])
        return {"idx": s["graph"], "out": s["out"]}
    if kind == "mrconv":
        update = api.mrconv_heads if c["heads"] else api.mrconv
        return {"out": update(x, s["idx"], s["W"], s["b"], keys=s.get("keys"), out=s["out"], ws=s["ws"])}
    if kind == "stage":
        y = api.max_pool_nodes(x, H, W, r, out=s["pooled"])
        return {"pooled": y, "out": api.linear(y, s["W"], s["b"], out=s["out"])}
    if kind == "stack":
        return {"out": s["la"].stack(x, H, W, s["W"], s["b"], _dilations(c), k, pool_r=r,
                                     schedule=SCHEDULE[c["schedule"]], ws=s["ws"], x_out=s["out"])}
    if kind == "vig_block":
        out, u = s["la"].vig_block(x, s["idx"], s["p"][0], s["ws"], u_out=s["u"], x_out=s["out"],
                                   idx_next=s["graph"], dilation_next=d, H=H, W=W, pool_r=r)
        # the graph was built on the handle's own stream
        torch.cuda.current_stream().wait_stream(s["la"].s_build)
        return {"out": out, "u": u, "idx": s["graph"]}
    return {"out": s["la"].vig_stack(x, s["p"], _dilations(c), k, schedule=SCHEDULE[c["schedule"]],
                                     ws=s["ws"], x_out=s["out"], H=H, W=W, pool_r=r)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    c = case
    kind, L, C, Co, k = c["kind"], c["L"], c["C"], c["Cout"], c["k"]
    es = 2 if c["dtype"] == "bf16" else 4
    R, RK = c["B"] * _nodes(c), c["B"] * _keys(c)
    x, graph = R * C * es, R * k * 4
    gram = 2.0 * R * _keys(c) * C
    if kind == "knn":
        return {"bytes": x + graph, "flops": gram}
    if kind == "stage":
        return {"bytes": x + RK * (C + Co) * es + C * Co * es, "flops": 2.0 * RK * C * Co}
    if kind in ("layer", "mrconv"):
        w = 2 * C * Co // (c["heads"] or 1)
        keys = RK * C * es if kind == "mrconv" and c["pool"] > 1 else 0
        return {"bytes": x + keys + graph + w * es + R * Co * es,
                "flops": 2.0 * R * w + (gram if kind == "layer" else 0)}
    if kind == "stack":
        # the first two blocks share a graph when their dilations are the same
        builds = L if L == 1 or len(set(_dilations(c)[:2])) > 1 else L - 1
        return {"bytes": 2 * x + L * 2 * C * C * es, "flops": builds * gram + L * 4.0 * R * C * C}
    fc = 12 * C * C  # FC1, the update, FC2 and the two layers of the FFN
    if kind == "vig_block":
        return {"bytes": 3 * x + 2 * graph + fc * es, "flops": gram + 2.0 * R * fc}
    builds = L if L == 1 or len(set(_dilations(c)[:2])) > 1 else L - 1
    return {"bytes": 2 * x + L * fc * es, "flops": builds * gram + L * 2.0 * R * fc}


# ---------------------------------------------------------------------------
# the definitions in float64; a tensor that the path stores (pooled keys, the
# max-relative half of an update's rows, a block's inner features) is rounded
# to the case's type there, as its definition says, and nothing else is
# ---------------------------------------------------------------------------
def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def _fc(x, w, b):
    y = x.reshape(-1, x.shape[-1]) @ w.t().contiguous()
    return (y if b is None else y + b).reshape(x.shape[:-1] + (w.shape[0],))


def _max_relative(x, idx, keys):
    """max over the neighbours t of keys[idx[.., t]] - x, without the edge tensor."""
    m = torch.full_like(x, -math.inf)
    for t in range(idx.shape[-1]):
        row = idx[:, :, t].long()[:, :, None].expand(-1, -1, x.shape[-1])
        m = torch.maximum(m, torch.gather(keys, 1, row))
    return m - x


def _update(x, idx, keys, w, b, stored, heads=0):
    m = stored(_max_relative(x, idx, keys))
    if not heads:
        return _fc(torch.cat([x, m], -1), w, b)
    hd = x.shape[-1] // heads
    y = torch.cat([_fc(torch.cat([x[..., h * hd:(h + 1) * hd], m[..., h * hd:(h + 1) * hd]], -1),
                       w[h], None) for h in range(heads)], -1)
    return y if b is None else y + b


def _block(x, u, idx, keys, p, stored):
    ut = stored(_gelu(_update(u, idx, keys, p["W_upd"], p["b_upd"], stored)))
    y = stored(_fc(ut, p["W_out"], p["b_out"]) + x)
    return _fc(stored(_gelu(_fc(y, p["W_1"], p["b_1"]))), p["W_2"], p["b_2"]) + y


def exact(case, seed):
    c = case
    kind, k, L = c["kind"], c["k"], c["L"]
    if kind == "knn" or L > 2:
        # graphs are ranks, which near-ties leave open; and a deeper stack's third
        # graph ranks features that hang on how a block was rounded, so its
        # outputs have no such value
        return None
    s = _data(c, seed)
    wide = lambda v: None if v is None else v.double()  # noqa: E731
    stored = lambda v: v.to(_dtype(c)).double()  # noqa: E731
    key = lambda v: stored(_pooled(v, c, "mean")) if c["pool"] > 1 else v  # noqa: E731
    x = s["x"].double()
    if kind == "layer":
        idx = _neighbours(x, key(x), k, c["d"])
        return {"idx": None, "out": _update(x, idx, key(x), wide(s["W"]), wide(s["b"]), stored)}
    if kind == "mrconv":
        keys = s["keys"].double() if "keys" in s else x
        return {"out": _update(x, s["idx"], keys, wide(s["W"]), wide(s["b"]), stored, c["heads"])}
    if kind == "stage":
        y = _pooled(x, c, "max")
        return {"pooled": y, "out": _fc(y, wide(s["W"]), wide(s["b"]))}
    dil = _dilations(c)
    if kind == "stack":
        # block l uses the graph of block l-1's input (blocks 0 and 1 that of x)
        src = x
        for l in range(L):
            idx = _neighbours(src, key(src), k, dil[l])
            y = _update(x, idx, key(x), wide(s["W"][l]), wide(s["b"][l]) if s["b"] is not None else None, stored)
            src, x = x, y if l + 1 == L else stored(y)
        return {"out": x}
    ps = [{n: wide(v) for n, v in p.items()} for p in s["p"]]
    if kind == "vig_block":
        u = _fc(x, ps[0]["W_in"], ps[0]["b_in"])
        us = stored(u)
        return {"out": _block(x, us, s["idx"], key(us), ps[0], stored), "u": u, "idx": None}
    src = None
    for l in range(L):
        u = stored(_fc(x, ps[l]["W_in"], ps[l]["b_in"]))
        src = u if src is None else src
        idx = _neighbours(src, key(src), k, dil[l])
        y = _block(x, u, idx, key(u), ps[l], stored)
        src, x = u, y if l + 1 == L else stored(y)
    return {"out": x}


def tolerance(case):
    """Four times the largest errors against `exact` measured over the listed and
    40 drawn cases:
      - without a graph of its own: 1.7e-3 (bf16, the outputs' rounding) and 4.7e-7
        (fp32), one value at most 1.3e-2 and 3.9e-6;
      - with one: near-ties that go the other way (1.4e-3 of the neighbours at
        most) change few rows by much: 6e-3 overall, one value by half;
      - from the third block of a stack on, the graphs rank features that carry
        the rounding of the blocks before: outputs that are alike only as far as
        those graphs are."""
    c = case
    bf16 = c["dtype"] == "bf16"
    if c["L"] > 2:
        return {"rel": 0.03, "max": 0.9, "differ": 0.006}
    if c["kind"] in ("layer", "knn", "stack", "vig_stack"):
        return {"rel": 0.024 if bf16 else 0.017, "max": 0.9, "differ": 0.006}
    if bf16:
        return {"rel": 0.007, "max": 0.05, "differ": 0.001}
    return {"rel": 2e-6, "max": 1.6e-5, "differ": 0.001}
