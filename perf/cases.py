"""What the performance of this library is measured on: attention over the tree-structured
KV cache of a PRM-guided search, through the public context calls, one case per way in
which a search program calls it.

A search keeps a tree of reasoning steps.  Between two prunings of the tree every generated
token costs, per layer, one decode call (and one append of the new K/V rows); every finished
step is scored by a reward model, which costs, per layer, one prefill call over the new steps'
tokens.  The plan is made once per search step and serves hundreds of tokens times the layers
of the model, so it belongs to what the program has in hand.

`path` of a case:
  decode    one layer's decode call
  step      one decode step of a few layers: per layer append the new rows, then attend; the
            plan has been advanced by a few tokens, as it is in the middle of a search step
  prefill   one layer's prefill call for the tokens of all leaf steps
`kv` is the pools' format (bf16, f32, or e4m3 codes with one scale per pool).  The tree is a
prompt of `prompt` tokens, `steps` search steps of `width` nodes whose parents are drawn from a
Dirichlet(`alpha`) distribution over the previous step's nodes (small: few parents survive,
much is shared; large: trajectories diverge), step lengths uniform in [`lo`, `hi`].
`searches` > 1 puts that many searches into one forest and one call.
"""
import functools
import math

import numpy as np
import torch

import paper_2502_13575_amd as ets

K_SCALE, V_SCALE = 0.0123, 0.0217  # scales of the e4m3 pools
Q_STD = 2.0      # scores spread by about two nats: softmax neither flat nor one-hot
ADVANCES = 5     # tokens into the search step that a "step" case stands


def _case(name, path, kv, kv_heads, group, head_dim, prompt, steps, lo, hi, width, alpha,
          topology, searches=1, layers=1, out_bf16=False):
    return {"name": name, "path": path, "kv": kv, "kv_heads": kv_heads, "group": group,
            "head_dim": head_dim, "prompt": prompt, "steps": steps, "lo": lo, "hi": hi,
            "width": width, "alpha": alpha, "topology": topology, "searches": searches,
            "layers": layers, "out_bf16": out_bf16}


def listed():
    return [
        # the smallest call there is: a handful of short steps, fp32 pools (launch latency)
        _case("tiny_f32", "decode", "f32", 1, 2, 64, 32, 3, 16, 16, 8, 1.0, 1001),
        # a narrow search on a 7B-shaped model (8 kv heads of 128, 4 query heads each)
        _case("w16", "decode", "bf16", 8, 4, 128, 512, 8, 64, 64, 16, 0.5, 1002),
        # width 64, trajectories that hardly share (a search that does not prune for sharing)
        _case("w64_divergent", "decode", "bf16", 8, 4, 128, 1024, 16, 128, 128, 64, 5.0, 1003),
        # the same search pruned for sharing, as one decode step of two layers with its appends
        _case("w64_pruned_step", "step", "bf16", 8, 4, 128, 1024, 16, 128, 128, 64, 0.2, 1003,
              layers=2),
        # an odd-sized search on a small model with heads of 64, bf16 results
        _case("w100_d64", "decode", "bf16", 8, 4, 64, 777, 20, 17, 150, 100, 0.5, 1007,
              out_bf16=True),
        # width 256 on a 34B-shaped model (8 query heads per kv head), ragged steps
        _case("w256_g8", "decode", "bf16", 8, 8, 128, 2048, 24, 32, 256, 256, 0.3, 1004),
        # the widest single search: long prompt, long ragged steps, 512 leaves
        _case("w512", "decode", "bf16", 8, 4, 128, 4096, 32, 64, 512, 512, 0.3, 1005),
        # the same search with the cache held in 8 bits
        _case("w512_e4m3", "decode", "e4m3", 8, 4, 128, 4096, 32, 64, 512, 512, 0.3, 1005),
        # a server's batch: sixteen searches of the 34B shape in one call, bf16 results
        _case("batch16_g8", "decode", "bf16", 8, 8, 128, 2048, 24, 32, 256, 256, 0.3, 1006,
              searches=16, out_bf16=True),
        # scoring the sixteen new steps of a narrow search
        _case("prefill_w16", "prefill", "bf16", 8, 4, 128, 512, 8, 64, 64, 16, 0.5, 1002),
        # scoring 64 new steps over an 8-bit cache
        _case("prefill_w64_e4m3", "prefill", "e4m3", 8, 4, 128, 1024, 16, 100, 150, 64, 0.2, 1003),
        # scoring 256 ragged steps on the 34B shape
        _case("prefill_w256_g8", "prefill", "bf16", 8, 8, 128, 2048, 24, 32, 256, 256, 0.3, 1004),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case anywhere in the ranges that the listed ones span, no dearer than the largest."""
    cap = {c["name"]: work(c) for c in listed() if c["name"] in ("batch16_g8", "prefill_w256_g8")}
    while True:
        path = rng.choice(["decode", "decode", "decode", "step", "prefill"])
        kv = rng.choice(["bf16", "bf16", "bf16", "bf16", "e4m3", "f32" if path == "decode" else "bf16"])
        d = 128 if path == "prefill" else rng.choice([128, 128, 128, 64])
        # fp32 pools are for checking a program's numbers: small searches only
        width = _log(rng, 8, 24 if kv == "f32" else 512)
        lo = _log(rng, 16, 64 if kv == "f32" else 128)
        c = _case("", path, kv, rng.choice([2, 4, 8, 8, 8]), rng.choice([1, 2, 4, 4, 8, 8]), d,
                  _log(rng, 32, 512 if kv == "f32" else 4096),
                  rng.randint(3, 8 if kv == "f32" else 32), lo, lo + rng.randint(0, 3 * lo), width,
                  round(math.exp(rng.uniform(math.log(0.2), math.log(5.0))), 3),
                  rng.randrange(1 << 30),
                  searches=rng.choice([1, 1, 1, _log(rng, 2, 16)]) if path == "decode" and kv != "f32" else 1,
                  layers=rng.randint(1, 4) if path == "step" else 1,
                  out_bf16=path == "decode" and rng.random() < 0.25)
        del c["name"]
        if c["width"] * c["searches"] * c["steps"] > 70000:
            continue
        w, most = work(c), cap["prefill_w256_g8" if path == "prefill" else "batch16_g8"]
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return c


# ---------------------------------------------------------------------------- the tree
class _Tree:
    pass


def _one_search(c, topology, room):
    """(parent, n_tokens, room, leaves) of one search; only nodes above a leaf are kept in the cache."""
    r = np.random.Generator(np.random.Philox(key=[int(topology), 11]))
    parent, prev = [np.array([-1])], np.array([0])
    n = 1
    for s in range(c["steps"]):
        if s == 0:
            par = np.zeros(c["width"], dtype=np.int64)
        else:
            p = np.maximum(r.dirichlet(np.full(prev.size, c["alpha"])), 1e-12)
            par = np.sort(prev[r.choice(prev.size, size=c["width"], p=p / p.sum())])
        parent.append(par)
        prev = np.arange(n, n + c["width"])
        n += c["width"]
    parent = np.concatenate(parent)
    length = r.integers(c["lo"], c["hi"] + 1, size=n)
    length[0] = c["prompt"]
    live = np.zeros(n, dtype=bool)
    live[prev] = True
    for i in range(n - 1, 0, -1):
        if live[i]:
            live[parent[i]] = True
    free = np.zeros(n, dtype=np.int64)
    free[prev] = room
    return parent, np.where(live, length, 0), free, prev


@functools.lru_cache(maxsize=64)
def _tree_of(key):
    c = dict(key)
    room = 4 * ADVANCES if c["path"] == "step" else 0
    parts, nodes = [], 0
    for s in range(c["searches"]):
        parent, length, free, leaves = _one_search(c, c["topology"] + 7919 * s, room)
        parts.append((np.where(parent < 0, -1, parent + nodes), length, free, leaves + nodes))
        nodes += parent.size
    t = _Tree()
    t.parent = np.concatenate([p[0] for p in parts]).astype(np.int32)
    t.length = np.concatenate([p[1] for p in parts]).astype(np.int32)
    rows = t.length.astype(np.int64) + np.concatenate([p[2] for p in parts])
    t.offset = np.cumsum(rows) - rows
    t.offset[rows == 0] = 0  # a step that was pruned away has no rows
    t.leaves = np.concatenate([p[3] for p in parts]).astype(np.int32)
    t.pool_tokens = int(rows.sum())
    return t


def _tree(c):
    return _tree_of(tuple(sorted((k, v) for k, v in c.items() if k != "name")))


def _chain(t, leaf):
    """Nodes from the root to the node of leaf query `leaf`."""
    nodes, x = [], int(t.leaves[leaf])
    while x >= 0:
        nodes.append(x)
        x = int(t.parent[x])
    return nodes[::-1]


def _lengths(c, t):
    """Rows of every node when the pass runs (a "step" case has been advanced)."""
    n = t.length.astype(np.int64)
    if c["path"] == "step":
        n[np.unique(t.leaves)] += ADVANCES
    return n


# --------------------------------------------------------------------------- the inputs
def _values(c, t, seed):
    """K, V [layer][kv head][pool row][D], Q, and for a "step" case the new rows K, V."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)
    dt = torch.float32 if c["kv"] == "f32" else torch.bfloat16
    hk, d, L = c["kv_heads"], c["head_dim"], t.leaves.size
    n_q = int(t.length[t.leaves].sum()) if c["path"] == "prefill" else L

    def pool(scale):
        if c["kv"] != "e4m3":
            return torch.empty((hk, t.pool_tokens, d), dtype=dt, device="cuda").normal_(generator=g)
        x = torch.empty((hk, t.pool_tokens, d), dtype=torch.float32, device="cuda")
        x.normal_(generator=g).div_(scale).clamp_(-448.0, 448.0)
        return x.to(torch.float8_e4m3fn).view(torch.uint8)

    k, v, q, k_new, v_new = [], [], [], [], []
    for _ in range(c["layers"]):
        k.append(pool(K_SCALE))
        v.append(pool(V_SCALE))
        q.append(torch.empty((n_q, hk * c["group"], d), dtype=torch.float32, device="cuda")
                 .normal_(std=Q_STD, generator=g).to(dt))
        if c["path"] == "step":
            x = torch.empty((2, L, hk, d), dtype=torch.float32, device="cuda").normal_(generator=g)
            if c["kv"] == "e4m3":
                x = torch.stack([x[0] / K_SCALE, x[1] / V_SCALE]).clamp_(-448.0, 448.0)
                x = x.to(torch.float8_e4m3fn).view(torch.uint8)
            else:
                x = x.to(dt)
            k_new.append(x[0].contiguous())
            v_new.append(x[1].contiguous())
    return k, v, q, k_new, v_new


def prepare(case, seed):
    t = _tree(case)
    k, v, q, k_new, v_new = _values(case, t, seed)
    ctx = ets.Context(case["kv_heads"], case["kv_heads"] * case["group"], case["head_dim"],
                      ets.ETS_F32 if case["kv"] == "f32" else ets.ETS_BF16, 0)
    if case["kv"] == "e4m3":
        ctx.set_kv_format(ets.ETS_KV_FP8_E4M3, K_SCALE, V_SCALE)
    if case["out_bf16"]:
        ctx.set_option("out_bf16", 1)
    ws = None
    if case["path"] == "prefill":
        ctx.plan_prefill(t.parent, t.offset, t.length, t.leaves)
    else:
        ctx.plan(t.parent, t.offset, t.length, t.leaves)
        for _ in range(ADVANCES if case["path"] == "step" else 0):
            ctx.plan_advance()
        ws = torch.empty(max(int(ctx.stats().workspace_bytes), 16), dtype=torch.uint8, device="cuda")
    n_q, hq = q[0].shape[0], q[0].shape[1]
    odt = torch.bfloat16 if case["out_bf16"] else torch.float32
    out = [torch.empty((n_q, hq, case["head_dim"]), dtype=odt, device="cuda") for _ in q]
    lse = [torch.empty((n_q, hq), dtype=torch.float32, device="cuda") for _ in q]
    return {"path": case["path"], "ctx": ctx, "rows": t.pool_tokens, "k": k, "v": v, "q": q,
            "k_new": k_new, "v_new": v_new, "out": out, "lse": lse, "ws": ws}


def run(state):
    ctx, rows, ws = state["ctx"], state["rows"], state["ws"]
    if state["path"] == "prefill":
        ctx.prefill(state["k"][0], state["v"][0], rows, state["q"][0], state["out"][0], state["lse"][0])
        return {"out": state["out"], "lse": state["lse"]}
    if state["path"] == "decode":
        ctx.decode(state["k"][0], state["v"][0], rows, state["q"][0], state["out"][0],
                   state["lse"][0], ws, ws.numel())
        return {"out": state["out"], "lse": state["lse"]}
    for i in range(len(state["k"])):
        ctx.kv_append(state["k"][i], state["v"][i], rows, state["k_new"][i], state["v_new"][i])
        ctx.decode(state["k"][i], state["v"][i], rows, state["q"][i], state["out"][i],
                   state["lse"][i], ws, ws.numel())
    return {"out": state["out"], "lse": state["lse"], "k_pool": state["k"], "v_pool": state["v"]}


# ------------------------------------------------------------ what is needed, what is right
def work(case):
    t = _tree(case)
    n = _lengths(case, t)
    hk, d = case["kv_heads"], case["head_dim"]
    hq = hk * case["group"]
    e = {"f32": 4, "bf16": 2, "e4m3": 1}[case["kv"]]
    e_q, e_o = 4 if case["kv"] == "f32" else 2, 2 if case["out_bf16"] else 4
    # rows on the way from the root to each node (the node's own included)
    path = n.copy()
    for i in range(1, path.size):
        if t.parent[i] >= 0:
            path[i] += path[t.parent[i]]
    own = n[t.leaves]
    if case["path"] == "prefill":
        n_q = int(own.sum())
        pairs = int((own * (path[t.leaves] - own) + own * (own + 1) // 2).sum())
    else:
        n_q = t.leaves.size
        pairs = int(path[t.leaves].sum())
    kv = 2 * int(n.sum()) * hk * d * e
    per_layer = kv + n_q * hq * (d * (e_q + e_o) + 4)
    if case["path"] == "step":
        per_layer += 4 * t.leaves.size * hk * d * e  # the new rows, read and written
    return {"bytes": case["layers"] * per_layer, "flops": case["layers"] * 4 * d * hq * pairs}


def tolerance(case):
    if case["kv"] == "f32":
        return {"rel": 1e-2 if case["out_bf16"] else 1e-5}
    # weights of 11 significant bits leave about 2e-4; a result in bf16 about 2e-3
    return {"rel": 1e-2 if case["out_bf16"] else 1e-3}


def exact(case, seed):
    t = _tree(case)
    if work(case)["flops"] > 3e13:
        return None
    k, v, q, k_new, v_new = _values(case, t, seed)
    n = _lengths(case, t)
    hk, g, d = case["kv_heads"], case["group"], case["head_dim"]
    scale = 1.0 / math.sqrt(d)
    first = {}  # the first leaf query of a node supplies its new row
    for l, node in enumerate(t.leaves.tolist()):
        first.setdefault(node, l)
    ks, vs = (K_SCALE, V_SCALE) if case["kv"] == "e4m3" else (1.0, 1.0)

    def wide(x, s):
        if x.dtype == torch.uint8:
            return x.view(torch.float8_e4m3fn).to(torch.float64) * float(np.float32(s))
        return x.to(torch.float64)

    outs, lses = [], []
    for i in range(case["layers"]):
        if case["path"] == "step":
            nodes = list(first)
            at = torch.tensor([int(t.offset[x] + n[x] - 1) for x in nodes], device="cuda")
            src = torch.tensor([first[x] for x in nodes], device="cuda")
            k[i][:, at] = k_new[i][src].transpose(0, 1)
            v[i][:, at] = v_new[i][src].transpose(0, 1)
        out = torch.zeros((q[i].shape[0], hk * g, d), dtype=torch.float64, device="cuda")
        lse = torch.full((q[i].shape[0], hk * g), -math.inf, dtype=torch.float64, device="cuda")
        row = 0
        for l in range(t.leaves.size):
            chain = _chain(t, l)
            at = np.concatenate([np.arange(t.offset[x], t.offset[x] + n[x]) for x in chain])
            at = torch.from_numpy(at).to("cuda")
            kk, vv = wide(k[i][:, at], ks), wide(v[i][:, at], vs)
            m = int(n[chain[-1]]) if case["path"] == "prefill" else 1
            qq = q[i][row:row + m].to(torch.float64).reshape(m, hk, g, d).permute(1, 0, 2, 3)
            s = torch.matmul(qq.reshape(hk, m * g, d), kk.transpose(1, 2).contiguous()) * scale
            if case["path"] == "prefill":  # token j of the step sees rows 0 .. j of it
                j = torch.arange(m, device="cuda")
                s.view(hk, m, g, -1)[..., -m:].masked_fill_((j[None, :] > j[:, None])[None, :, None, :],
                                                            -math.inf)
            z = torch.logsumexp(s, dim=-1)
            o = torch.matmul(torch.exp(s - z[..., None]), vv)
            out[row:row + m] = o.reshape(hk, m, g, d).permute(1, 0, 2, 3).reshape(m, hk * g, d)
            lse[row:row + m] = z.reshape(hk, m, g).permute(1, 0, 2).reshape(m, hk * g)
            row += m
        outs.append(out)
        lses.append(lse)
    if case["path"] == "step":
        return {"out": outs, "lse": lses, "k_pool": k, "v_pool": v}
    return {"out": outs, "lse": lses}
