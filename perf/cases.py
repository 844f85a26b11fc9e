"""The work a program that serves a model over KVMem has this library do, as timed cases.

Every case goes through the functions of `paper_2609_04852_amd.kvmem` with device
buffers that the program already holds: paged K/V pools, the block table, the
Mean-K index, view tables, workspaces.  Sizes are those of `workload.CONFIGS`
where that has them.  Kinds of work:

  step         one layer of a decode step: selection, then attention over the view
  recall       a recall point's selection: every layer, every query token of a prefill
  attn         a prefill's query tokens replayed over a view that is already chosen
  index        Mean-K index of a range of blocks (prefill: all; later: the new ones)
  index_rope   the same from keys that carry RoPE
  working_set  a recall point's update of the bounded execution pool
  materialize  a view's K re-encoded at compact positions, V copied

Inputs are drawn on the GPU with the recipe of `workload.py`: keys and values
N(0, 1) around a per-(page, KV head) offset, a few blocks aligned with the
queries, or keys around 256 centres with Zipf weights ("mixture").
"""
import math

import numpy as np
import torch

from paper_2609_04852_amd import kvmem as K

ROPE_BASE = 1e6
DTYPES = {"bf16": (torch.bfloat16, K.KVMEM_BF16, 2), "f32": (torch.float32, K.KVMEM_F32, 4),
          "fp8": (torch.float8_e4m3fn, K.KVMEM_FP8_E4M3, 1)}
CHUNK = 1 << 26  # elements drawn at a time


def _case(name, kind, **kw):
    base = dict(kind=kind, hkv=8, group=4, d=128, bt=16, dtype="bf16", blocks=4096, sink=0, recent=64, view=512,
                n_q=1, layers=1, mode="mean", keys="offset", last=0, first=0)
    base.update(kw)
    if name:
        base["name"] = name
    return base


def listed():
    return [
        # the smallest configuration there is: what a call costs at all
        _case("step_tiny_f32", "step", hkv=1, d=64, dtype="f32", blocks=256, recent=4, view=36),
        # a decode step of one layer of an 8x4 GQA model over 64K, 256K and 1M tokens of history
        _case("step_64k", "step", blocks=4096, recent=64, view=512),
        _case("step_256k", "step", blocks=16384, recent=256, view=2048, last=5),
        _case("step_1m", "step", blocks=65536, recent=512, view=16384),
        # the 1M step on an FP8 cache
        _case("step_1m_fp8", "step", dtype="fp8", blocks=65536, recent=512, view=16384),
        # a layer of a speculative decode step: 4 query tokens, one selection per KV head, 64-token blocks
        _case("step_1m_mtp4", "step", bt=64, blocks=16384, recent=128, view=4096, n_q=4, mode="max", keys="mixture"),
        # a recall point: 4 layers, a 128-token prefill, one selection for all of them
        _case("recall_1m", "recall", bt=32, blocks=32768, recent=256, view=2048, n_q=128, layers=4),
        # that prefill's attention over the 64K view of one layer, the last page half full
        _case("prefill_attn_64k", "attn", bt=32, blocks=4096, view=2048, n_q=128, last=17),
        # the index of a 1M-token history, at load time
        _case("index_1m", "index", blocks=65536),
        # the index of the blocks that a 32K-token prefill adds to a history, from keys with RoPE
        _case("index_rope_32k", "index_rope", blocks=18331, first=16283),
        # a recall point's working-set update: a 64K view over a pool of 80K tokens
        _case("working_set_64k", "working_set", bt=32, blocks=32768, view=2048),
        # a 128K view laid out anew
        _case("materialize_128k", "materialize", bt=32, blocks=32768, view=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 8 + ["attn"] * 3 + ["recall"] * 2 + ["index", "index_rope", "working_set", "materialize"])
    c = _case(None, kind)
    c["hkv"] = rng.choice([1, 2, 4, 8, 8])
    c["group"] = rng.choice([1, 2, 4, 4, 5, 7, 8])
    c["d"] = rng.choice([64, 128, 128])
    c["bt"] = rng.choice([16, 32, 64])
    c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "fp8", "f32"])
    if kind in ("working_set", "materialize") and c["dtype"] == "fp8":
        c["dtype"] = "bf16"  # FP8 keys are not re-encoded
    # at most the 1M-token history of the listed cases, and their K/V bytes
    most = min(1 << 20, (1 << 31) // (c["hkv"] * c["d"] * DTYPES[c["dtype"]][2]))
    tokens = _log_int(rng, 4096, most)
    c["blocks"] = max(40, tokens // c["bt"])
    c["sink"] = rng.choice([0, 0, 1, 4])
    c["recent"] = max(1, min(c["blocks"] // 8, _log_int(rng, 64, 8192) // c["bt"]))
    c["view"] = c["sink"] + c["recent"] + max(1, int((c["blocks"] - c["sink"] - c["recent"]) * rng.uniform(0.03, 0.3)))
    c["last"] = rng.choice([0, rng.randint(1, c["bt"])])
    c["keys"] = rng.choice(["offset", "offset", "mixture"])
    if kind == "step":
        c["n_q"] = rng.choice([1, 1, 2, 4])
        c["mode"] = rng.choice(["mean", "mean", "max"])
    elif kind == "recall":
        c["layers"] = rng.randint(1, 4)
        c["n_q"] = _log_int(rng, 16, 128)
        c["mode"] = rng.choice(["mean", "mean", "max"])
        c["dtype"] = "bf16"
        c["blocks"] = min(c["blocks"], 32768)
        c["recent"] = min(c["recent"], c["blocks"] // 8)
        c["view"] = c["sink"] + c["recent"] + c["blocks"] // 16
    elif kind == "attn":
        c["n_q"] = _log_int(rng, 8, 128)
        c["view"] = max(8, min(c["blocks"], 65536 // c["bt"], c["view"]))
    elif kind in ("index", "index_rope"):
        c["first"] = rng.choice([0, rng.randint(0, c["blocks"] - 1)])
    else:
        c["view"] = min(c["view"], 65536 // c["bt"])
    # no more work than the listed prefill and recall; less on fp32 pools, which are for checks, not for prefills
    most = 1.2e11 if c["dtype"] != "f32" else 8e9
    while work(c)["flops"] > most and c["n_q"] > 1:
        c["n_q"] = c["n_q"] * 2 // 3
    return c


def _geom(c):
    scale = _scale(c)
    return K.Geom(c["hkv"], c["hkv"] * c["group"], c["d"], c["bt"], DTYPES[c["dtype"]][1], scale, scale)


def _scale(c):
    return float(np.float32((8 if c["keys"] == "offset" else 16) / 448)) if c["dtype"] == "fp8" else 1.0


# ---- inputs ---------------------------------------------------------------

def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt * 7919) % (1 << 62))
    return g


def _store(x, c):
    if c["dtype"] == "fp8":
        return (x / _scale(c)).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
    return x.to(DTYPES[c["dtype"]][0])


def _chunks(c):
    per = max(1, CHUNK // (c["hkv"] * c["bt"] * c["d"]))
    return [(lo, min(c["blocks"], lo + per)) for lo in range(0, c["blocks"], per)]


def _pool(c, seed, salt, mixture=False):
    """[blocks][hkv][bt][d] (one page per block)."""
    g = _gen(seed, salt)
    pool = torch.empty((c["blocks"], c["hkv"], c["bt"], c["d"]), dtype=DTYPES[c["dtype"]][0], device="cuda")
    if mixture:
        centres = torch.randn((c["hkv"], 256, c["d"]), generator=g, device="cuda") * 2
        w = torch.arange(1, 257, device="cuda", dtype=torch.float32) ** -1.1
        pick = torch.multinomial(w, c["blocks"] * c["hkv"], replacement=True, generator=g).view(c["blocks"], c["hkv"])
        heads = torch.arange(c["hkv"], device="cuda")
    for lo, hi in _chunks(c):
        x = torch.randn((hi - lo, c["hkv"], c["bt"], c["d"]), generator=g, device="cuda")
        if mixture:
            x += centres[heads, pick[lo:hi]][:, :, None, :]
        else:
            x += torch.randn((hi - lo, c["hkv"], 1, c["d"]), generator=g, device="cuda") * 0.5
        pool[lo:hi] = _store(x, c)
    return pool


def _queries(c, seed):
    """[layers][n_q][Hq][d]: per KV head a direction, per query N(0, 0.5^2) around it."""
    g = _gen(seed, 1)
    u = torch.randn((c["layers"], 1, c["hkv"], 1, c["d"]), generator=g, device="cuda")
    e = torch.randn((c["layers"], c["n_q"], c["hkv"], c["group"], c["d"]), generator=g, device="cuda")
    return (u + 0.5 * e).reshape(c["layers"], c["n_q"], c["hkv"] * c["group"], c["d"]).contiguous()


def _plant(c, seed, pool, q, b2p):
    """A few candidate blocks' keys aligned with the mean query of their KV head (cosine 0.9)."""
    g = _gen(seed, 2)
    n_cand = c["blocks"] - c["sink"] - c["recent"]
    n = max(1, min(n_cand // 4, c["blocks"] // 256))
    ids = c["sink"] + torch.randperm(n_cand, generator=g, device="cuda")[:n]
    u = q.view(c["n_q"], c["hkv"], c["group"], c["d"]).mean((0, 2))
    u = u / u.norm(dim=-1, keepdim=True)
    nu = torch.randn((n, c["hkv"], c["bt"], c["d"]), generator=g, device="cuda")
    u = u[None, :, None, :]
    nu = nu - (nu * u).sum(-1, keepdim=True) * u
    nu = nu / nu.norm(dim=-1, keepdim=True)
    pool[b2p[ids].long()] = _store(math.sqrt(c["d"]) * (0.9 * u + math.sqrt(0.19) * nu), c)


def _table(c, seed, salt=3):
    return torch.randperm(c["blocks"], generator=_gen(seed, salt), device="cuda").to(torch.int32)


def _keys(c, seed, layer, q, b2p):
    pool = _pool(c, seed, 10 + layer, c["keys"] == "mixture")
    if c["keys"] == "offset" and layer == 0:
        _plant(c, seed, pool, q[0], b2p)
    return pool


def _angles(c, pos):
    """[n][bt][d/2] of blocks whose first tokens sit at pos, in 64 bits."""
    f = ROPE_BASE ** (-2.0 * torch.arange(c["d"] // 2, device="cuda", dtype=torch.float64) / c["d"])
    return (pos[:, None] + torch.arange(c["bt"], device="cuda"))[:, :, None].double() * f


def _turn(x, a):
    """x [n][hkv][bt][d] turned by the angles a [n][bt][d/2] (rotate-half form)."""
    h = x.shape[-1] // 2
    cos, sin = a.cos()[:, None].to(x.dtype), a.sin()[:, None].to(x.dtype)
    return torch.cat([x[..., :h] * cos - x[..., h:] * sin, x[..., :h] * sin + x[..., h:] * cos], -1)


def _encoded_pool(c, seed, b2p):
    """A key pool whose blocks carry RoPE at their own positions b * bt + t."""
    pool = _pool(c, seed, 10)
    for lo, hi in _chunks(c):
        pages = b2p[lo:hi].long()
        x = _values(c, pool[pages], torch.float32)
        pool[pages] = _store(_turn(x, _angles(c, torch.arange(lo, hi, device="cuda") * c["bt"])), c)
    return pool


def _views(c, seed):
    """Four recalls' views: each keeps about three quarters of the one before."""
    r = np.random.default_rng(seed)
    views, prev = [], np.sort(r.choice(c["blocks"], c["view"], replace=False))
    for _ in range(4):
        views.append(torch.from_numpy(prev.astype(np.int32)).cuda())
        keep = r.choice(prev, (3 * c["view"]) // 4, replace=False)
        rest = np.setdiff1d(np.arange(c["blocks"]), keep)
        prev = np.sort(np.concatenate([keep, r.choice(rest, c["view"] - len(keep), replace=False)]))
    return views


def _exec_pages(c):
    return c["view"] + max(1, c["view"] // 4)


# ---- the calls --------------------------------------------------------------

def prepare(case, seed):
    c = case
    g = _geom(c)
    s = {"c": c, "g": g, "b2p": _table(c, seed)}
    mode = K.KVMEM_REDUCE_MEAN_ALL if c["mode"] == "mean" else K.KVMEM_REDUCE_MAX_GROUP
    i32 = dict(dtype=torch.int32, device="cuda")
    if c["kind"] in ("step", "recall"):
        s["mode"] = mode
        s["budget"] = c["view"] * c["bt"]
        s["q"] = _queries(c, seed)
        per_layer = K.kvmem_index_bytes(g, c["blocks"]) // 4
        s["index"] = torch.empty(c["layers"] * per_layer, dtype=torch.float32, device="cuda")
        for l in range(c["layers"]):
            pool = _keys(c, seed, l, s["q"], s["b2p"])
            K.kvmem_build_index(g, pool, s["b2p"], 0, c["blocks"], s["index"][l * per_layer:(l + 1) * per_layer])
        n_sel = s["n_sel"] = 1 if c["mode"] == "mean" else c["layers"] * c["hkv"]
        s["vb"] = torch.empty((n_sel, c["view"]), **i32)
        s["vp"] = torch.empty((n_sel, c["view"]), **i32)
        s["ws"] = torch.empty(K.kvmem_select_workspace_bytes(g, c["layers"], c["n_q"], c["blocks"], c["sink"],
                                                             c["recent"], mode), dtype=torch.uint8, device="cuda")
        if c["kind"] == "recall":
            s["scores"] = torch.empty((n_sel, c["blocks"]), dtype=torch.float32, device="cuda")
        else:
            s["k"], s["v"] = pool, _pool(c, seed, 50)
    elif c["kind"] == "attn":
        s["n_sel"] = 1
        s["q"] = _queries(c, seed)
        s["k"], s["v"] = _keys(dict(c, recent=0), seed, 0, s["q"], s["b2p"]), _pool(c, seed, 50)
        s["vp"] = _attn_view(c, seed, s["b2p"])
    elif c["kind"] in ("index", "index_rope"):
        s["k"] = _pool(c, seed, 10) if c["kind"] == "index" else _encoded_pool(c, seed, s["b2p"])
        s["index"] = torch.zeros(K.kvmem_index_bytes(g, c["blocks"]) // 4, dtype=torch.float32, device="cuda")
    elif c["kind"] == "working_set":
        s["k"], s["v"], s["views"] = _pool(c, seed, 10), _pool(c, seed, 50), _views(c, seed)
        n = _exec_pages(c)
        s["set"] = K.WorkingSetArrays(c["blocks"], n)
        s["set"].reset()
        s["ke"] = torch.zeros((n,) + tuple(s["k"].shape[1:]), dtype=s["k"].dtype, device="cuda")
        s["ve"] = torch.zeros_like(s["ke"])
        s["pages"] = torch.empty(c["view"], **i32)
        s["counts"] = torch.zeros(16, **i32)
        s["ws"] = torch.empty(K.kvmem_working_set_workspace_bytes(c["view"], n), dtype=torch.uint8, device="cuda")
        s["at"] = 0
        run(s)  # the first recall, which finds the pool empty
    else:
        s["k"], s["v"] = _pool(c, seed, 10), _pool(c, seed, 50)
        s["src"] = s["b2p"][torch.sort(_table(c, seed, 4)[: c["view"]])[0].long()].contiguous()
        s["dst"] = torch.randperm(c["view"], generator=_gen(seed, 5), device="cuda").to(torch.int32)
        s["pos"] = torch.arange(c["view"], device="cuda", dtype=torch.int64) * c["bt"]
        s["ke"] = torch.zeros((c["view"],) + tuple(s["k"].shape[1:]), dtype=s["k"].dtype, device="cuda")
        s["ve"] = torch.zeros_like(s["ke"])
    if c["kind"] in ("step", "attn"):
        s["aws"] = torch.empty(K.kvmem_sparse_attn_workspace_bytes(g, c["n_q"], s["n_sel"], c["view"]),
                               dtype=torch.uint8, device="cuda")
        s["out"] = torch.empty(tuple(s["q"].shape[1:]), dtype=torch.float32, device="cuda")
        s["lse"] = torch.empty((c["n_q"], c["hkv"] * c["group"]), dtype=torch.float32, device="cuda")
    return s


def _attn_view(c, seed, b2p):
    ids = torch.sort(_table(c, seed, 4)[: c["view"]])[0]
    return b2p[ids.long()].contiguous().view(1, -1)


def run(s):
    c, g = s["c"], s["g"]
    kind = c["kind"]
    if kind in ("step", "recall"):
        K.kvmem_select(g, s["q"], s["index"], c["blocks"], c["sink"], c["recent"], s["budget"], s["budget"], s["mode"],
                       0.0, s["b2p"], s["vb"], s["vp"], s["ws"], s.get("scores"))
        if kind == "recall":
            return {"blocks": s["vb"], "pages": s["vp"], "scores": s["scores"]}
    if kind in ("step", "attn"):
        K.kvmem_sparse_attn(g, s["q"][0], s["k"], s["v"], s["vp"], s["n_sel"], c["view"], c["last"] or c["bt"], 0.0,
                            s["out"], s["aws"], s["lse"])
        got = {"out": s["out"], "lse": s["lse"]}
        return got if kind == "attn" else dict(got, blocks=s["vb"], pages=s["vp"])
    if kind == "index":
        K.kvmem_build_index(g, s["k"], s["b2p"], c["first"], c["blocks"] - c["first"], s["index"])
        return s["index"]
    if kind == "index_rope":
        K.kvmem_build_index_rope(g, s["k"], s["b2p"], c["first"], c["blocks"] - c["first"], s["index"], ROPE_BASE)
        return s["index"]
    if kind == "working_set":
        K.kvmem_working_set_update(g, ROPE_BASE, s["set"], s["at"], s["views"][s["at"] % 4], 0, 8, s["b2p"], s["k"],
                                   s["v"], s["ke"], s["ve"], s["pages"], s["counts"], s["ws"])
        s["at"] += 1
        return {"pages": s["pages"], "counts": s["counts"], "k": s["ke"], "v": s["ve"]}
    K.kvmem_materialize(g, ROPE_BASE, s["k"], s["v"], s["src"], s["pos"], s["dst"], s["ke"], s["ve"])
    return {"k": s["ke"], "v": s["ve"]}


# ---- what a pass cannot do without ------------------------------------------

def work(case):
    c = case
    e = DTYPES[c["dtype"]][2]
    rows, cand = c["group"] * c["n_q"], c["blocks"] - c["sink"] - c["recent"]
    head = c["hkv"] * c["d"]
    n_sel = 1 if c["mode"] == "mean" else c["layers"] * c["hkv"]
    select = {"bytes": 4 * c["layers"] * (cand * head + rows * head) + 4 * c["blocks"] + 8 * n_sel * c["view"],
              "flops": 2 * c["layers"] * cand * rows * head}
    attn = {"bytes": 2 * c["view"] * c["bt"] * head * e + 4 * c["view"] + 8 * rows * head,
            "flops": 4 * c["view"] * c["bt"] * rows * head}
    if c["kind"] == "step":
        return {k: select[k] + attn[k] for k in select}
    if c["kind"] == "recall":
        return dict(select, bytes=select["bytes"] + 4 * n_sel * c["blocks"])
    if c["kind"] == "attn":
        return attn
    n, block = c["blocks"] - c["first"], c["bt"] * head
    if c["kind"] in ("index", "index_rope"):
        return {"bytes": n * (block * e + 4 * head), "flops": n * block * (1 if c["kind"] == "index" else 4)}
    if c["kind"] == "working_set":
        # a quarter of the view is loaded (K and V read and written); K of most of the rest is turned in place
        return {"bytes": c["view"] * block * e * (0.25 * 4 + 0.75 * 2), "flops": c["view"] * block * 3}
    return {"bytes": 4 * c["view"] * block * e, "flops": c["view"] * block * 3}


def tolerance(case):
    """About four times what the outputs were off the 64-bit result (relative, in the 2-norm)."""
    kind, dtype = case["kind"], case["dtype"]
    if kind == "index":
        return "exact"  # the sums are exact and rounded once
    if kind == "index_rope":
        return {"rel": 3e-7}  # 6e-8
    if kind in ("working_set", "materialize"):  # re-encoded keys, rounded to the pool's type: 2e-3, fp32 7e-8
        return {"rel": 8e-3, "max": 5e-2} if dtype == "bf16" else {"rel": 3e-7}
    if kind == "recall":
        return {"rel": 1e-6, "differ": 0.01}  # 3e-8 (mean) to 2e-7 (max)
    return {"rel": 2e-5, "differ": 0.01}  # 1e-6 to 5e-6 (out; clustered keys the most)


# ---- the same in 64 bits ------------------------------------------------------

def _values(c, x, dtype=torch.float64):
    return x.to(dtype) * _scale(c) if c["dtype"] == "fp8" else x.to(dtype)


def _means(c, pool, b2p):
    """[blocks][hkv][d]: block means in 64 bits."""
    out = torch.empty((c["blocks"], c["hkv"], c["d"]), dtype=torch.float64, device="cuda")
    for lo, hi in _chunks(c):
        out[lo:hi] = _values(c, pool[b2p[lo:hi].long()]).mean(2)
    return out


def _exact_relevance(c, q, means, acc):
    """Adds one layer's [n_sel of the layer][candidates] to acc (a list)."""
    lo, hi = c["sink"], c["blocks"] - c["recent"]
    for h in range(c["hkv"]):
        rows = q[:, h * c["group"]:(h + 1) * c["group"]].reshape(-1, c["d"]).double() / math.sqrt(c["d"])
        p = torch.softmax(rows @ means[lo:hi, h].T.contiguous(), -1)
        if c["mode"] == "max":
            acc.append(p.max(0)[0])
        elif acc:
            acc[0] += p.sum(0)
        else:
            acc.append(p.sum(0))


def _exact_attn(c, q, k, v, vp):
    hq = c["hkv"] * c["group"]
    out = torch.empty((c["n_q"], hq, c["d"]), dtype=torch.float64, device="cuda")
    lse = torch.empty((c["n_q"], hq), dtype=torch.float64, device="cuda")
    n_tok = c["view"] * c["bt"] - (c["bt"] - (c["last"] or c["bt"]))
    for h in range(c["hkv"]):
        pages = vp[h if vp.shape[0] > 1 else 0].long()
        kt = _values(c, k[pages, h]).reshape(-1, c["d"])[:n_tok]
        vt = _values(c, v[pages, h]).reshape(-1, c["d"])[:n_tok]
        at = slice(h * c["group"], (h + 1) * c["group"])
        s = (q[:, at].reshape(-1, c["d"]).double() / math.sqrt(c["d"])) @ kt.T.contiguous()
        lse[:, at] = torch.logsumexp(s, -1).view(c["n_q"], -1)
        out[:, at] = (torch.softmax(s, -1) @ vt).view(c["n_q"], -1, c["d"])
    return {"out": out, "lse": lse}


def exact(case, seed):
    c = case
    b2p = _table(c, seed)
    if c["kind"] in ("step", "recall"):
        q, rel = _queries(c, seed), []
        for l in range(c["layers"]):
            k = _keys(c, seed, l, q, b2p)
            _exact_relevance(c, q[l], _means(c, k, b2p), rel)
        rel = torch.stack(rel) / (c["layers"] * c["hkv"] * c["group"] if c["mode"] == "mean" else 1)
        if c["kind"] == "recall":
            scores = torch.full((rel.shape[0], c["blocks"]), math.inf, dtype=torch.float64, device="cuda")
            scores[:, c["sink"]:c["blocks"] - c["recent"]] = rel
            return {"blocks": None, "pages": None, "scores": scores}
        n = c["view"] - c["sink"] - c["recent"]
        top = torch.sort(rel, dim=1, descending=True, stable=True)[1][:, :n]
        ids = torch.arange(c["blocks"], device="cuda").expand(rel.shape[0], -1)
        view = torch.cat([ids[:, :c["sink"]], torch.sort(top, 1)[0] + c["sink"], ids[:, c["blocks"] - c["recent"]:]], 1)
        return dict(_exact_attn(c, q[0], k, _pool(c, seed, 50), b2p[view]), blocks=None, pages=None)
    if c["kind"] == "attn":
        q = _queries(c, seed)
        k = _keys(dict(c, recent=0), seed, 0, q, b2p)
        return _exact_attn(c, q[0], k, _pool(c, seed, 50), _attn_view(c, seed, b2p))
    if c["kind"] in ("index", "index_rope"):
        k = _pool(c, seed, 10) if c["kind"] == "index" else _encoded_pool(c, seed, b2p)
        tiles = -(-c["blocks"] // 64)
        rows = torch.zeros((tiles * 64, c["hkv"], c["d"]), dtype=torch.float64, device="cuda")
        for lo, hi in _chunks(c):
            lo = max(lo, c["first"])
            if lo >= hi:
                continue
            x = _values(c, k[b2p[lo:hi].long()])
            if c["kind"] == "index_rope":
                x = _turn(x, -_angles(c, torch.arange(lo, hi, device="cuda") * c["bt"]))
            rows[lo:hi] = x.mean(2)
        return rows.view(tiles, 64, c["hkv"], c["d"] // 4, 4).permute(0, 2, 3, 1, 4).reshape(-1)
    k, v = _pool(c, seed, 10), _pool(c, seed, 50)
    if c["kind"] == "materialize":
        src = b2p[torch.sort(_table(c, seed, 4)[: c["view"]])[0].long()]
        dst = torch.randperm(c["view"], generator=_gen(seed, 5), device="cuda")
        return _placed(c, k, v, c["view"], src, dst, torch.arange(c["view"], device="cuda") * c["bt"])
    # the second recall: misses take the pages that hold no selected block, in order after the first view's pages
    n, views = _exec_pages(c), [x.tolist() for x in _views(c, seed)[:2]]
    block = {p: b for p, b in enumerate(views[0])}
    pos = {p: p * c["bt"] for p in block}
    page = {b: p for p, b in block.items()}
    hits = {page[b] for b in views[1] if b in page}
    free = [p for p in ((c["view"] + i) % n for i in range(n)) if p not in hits]
    for i, b in enumerate(views[1]):
        p = page[b] if b in page else free.pop(0)
        block[p], pos[p] = b, i * c["bt"]
    dst = torch.tensor(sorted(block), device="cuda")
    src = b2p[torch.tensor([block[p] for p in sorted(block)], device="cuda")]
    return dict(_placed(c, k, v, n, src, dst, torch.tensor([pos[p] for p in sorted(block)], device="cuda")),
                pages=None, counts=None)


def _placed(c, k, v, n, src, dst, pos):
    """Pools of n pages: page dst[i] holds K of page src[i] turned to pos[i], and its V."""
    ke = torch.zeros((n,) + tuple(k.shape[1:]), dtype=torch.float64, device="cuda")
    ve = torch.zeros_like(ke)
    for lo in range(0, len(src), 512):
        at, to = src[lo:lo + 512].long(), dst[lo:lo + 512].long()
        ke[to] = _turn(k[at].double(), _angles(c, pos[lo:lo + 512]))
        ve[to] = v[at].double()
    return {"k": ke, "v": ve}
