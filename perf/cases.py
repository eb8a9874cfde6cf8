"""Cases of the decoding step's hot path, timed through the public entry points.

A case is a dict of plain sizes.  Its "kind" names the work:

  step     attention, top-k and verify + expand of one fp32 step (the small
           reference configuration: launches and latency)
  layer    one attention layer of a single sequence: rotary embedding of the
           tree rows in place, then tree attention
  attn     tree attention alone: one long sequence, a padded batch whose
           sequences have their own lengths and tree sizes, decode-sized calls
           (one to four nodes), trees of more than 128 nodes; caches contiguous
           or paged, bf16 or E4M3
  topk     argmax and top-k of the verification logits
  sample   sampling verification of the tree
  update   the bookkeeping after verification: verify + expand, commit of the
           accepted rows, stepping, merge into the candidate pool, retrieval

Buffers that a decoding loop keeps (outputs, workspaces, the pool) are made in
prepare(); run() makes the calls of one pass.
"""
import math
import random

import numpy as np
import torch

import paper_2607_10661_amd as P

DEV = "cuda:0"
LOGIT_STD = math.sqrt(2.0)


def listed():
    return [
        # the smallest: the fp32 reference configuration, one whole step
        dict(name="step_tiny_f32", kind="step", Hq=2, Hkv=2, D=64, T=16, kv=128, V=1000, k=4),
        # batch 1, multi-head attention: an interactive session, per layer
        dict(name="layer_7b", kind="layer", Hq=32, Hkv=32, D=128, T=64, kv=2048),
        # batch 1, grouped queries, a long document as context
        dict(name="attn_long", kind="attn", B=1, Hq=32, Hkv=8, D=128, T=64, kv_lo=32768,
             kv_hi=32768, lens=0, page=0, f8=False, ragged=False),
        # a serving batch: sequences of very different lengths, trees of their own sizes
        dict(name="attn_batch", kind="attn", B=16, Hq=32, Hkv=8, D=128, T=64, kv_lo=512,
             kv_hi=8192, lens=4, page=0, f8=False, ragged=True),
        # the same batch on paged caches, as serving engines keep them
        dict(name="attn_paged", kind="attn", B=16, Hq=32, Hkv=8, D=128, T=64, kv_lo=512,
             kv_hi=8192, lens=4, page=64, f8=False, ragged=False),
        # fewer, longer sequences on 8-bit pages
        dict(name="attn_paged_fp8", kind="attn", B=6, Hq=32, Hkv=8, D=128, T=48, kv_lo=1024,
             kv_hi=16384, lens=7, page=128, f8=True, ragged=True),
        # decode-sized calls: the step in which no tree was found
        dict(name="attn_decode", kind="attn", B=16, Hq=32, Hkv=8, D=128, T=1, kv_lo=8192,
             kv_hi=8192, lens=0, page=0, f8=False, ragged=False),
        # a wide tree: masks no longer fit two words per node
        dict(name="attn_big_tree", kind="attn", B=2, Hq=32, Hkv=8, D=128, T=256, kv_lo=1000,
             kv_hi=4096, lens=1, page=0, f8=False, ragged=False),
        # the largest: logits of a batch's nodes over a large vocabulary
        dict(name="topk_batch", kind="topk", R=1040, V=128256, k=8, f32=False),
        # one sequence, a vocabulary with a few added tokens: rows start at odd addresses
        dict(name="topk_odd_rows", kind="topk", R=65, V=32003, k=4, f32=False),
        # sampling instead of greedy verification, the same logits
        dict(name="sample_batch", kind="sample", B=16, T=64, V=128256, temp=1.0),
        # host-free bookkeeping between two forward passes
        dict(name="tree_update", kind="update", B=16, Hkv=8, D=128, T=64, V=32000, k=4,
             e_max=2048),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "layer", "long", "batch", "paged", "fp8", "decode", "big_tree",
                       "topk", "topk", "sample", "update"])
    if kind == "step":
        Hkv = rng.choice([1, 2, 4])
        return dict(kind="step", Hq=Hkv * rng.choice([1, 2]), Hkv=Hkv, D=rng.choice([64, 128]),
                    T=rng.randint(4, 64), kv=_log(rng, 32, 512), V=_log(rng, 500, 32000), k=4)
    if kind == "layer":
        Hq, Hkv = rng.choice([(32, 32), (40, 40), (32, 8)])
        return dict(kind="layer", Hq=Hq, Hkv=Hkv, D=rng.choice([64, 128, 128]),
                    T=rng.randint(8, 128), kv=_log(rng, 256, 8192))
    c = dict(kind="attn", B=1, Hq=32, Hkv=8, D=128, T=64, kv_lo=0, kv_hi=0,
             lens=rng.randint(0, 10 ** 6), page=0, f8=False, ragged=False)
    if kind == "long":
        c["kv_lo"] = c["kv_hi"] = _log(rng, 4096, 32768)
        c["T"] = rng.randint(1, 96)
        return c
    if kind in ("batch", "paged", "fp8"):
        c["B"] = _log(rng, 2, 64)
        c["kv_hi"] = min(16384 if kind == "fp8" else 8192, _log(rng, 512, 131072 // c["B"]))
        c["kv_lo"] = max(16, c["kv_hi"] // rng.choice([2, 8, 16]))
        c["T"] = rng.randint(16, 64)
        c["ragged"] = rng.random() < 0.5
        c["Hkv"] = rng.choice([8, 8, 4])
        if kind != "batch":
            c["page"] = rng.choice([32, 64, 128])
        c["f8"] = kind == "fp8"
        return c
    if kind == "decode":
        c["B"] = _log(rng, 1, 32)
        c["kv_hi"] = _log(rng, 1024, min(32768, 131072 // c["B"]))
        c["kv_lo"] = max(512, c["kv_hi"] // rng.choice([1, 4]))
        c["T"] = rng.randint(1, 4)
        c["Hkv"] = rng.choice([8, 8, 32]) if c["B"] * c["kv_hi"] <= 32768 else 8
        c["page"] = rng.choice([0, 0, 64])
        return c
    if kind == "big_tree":
        c["B"] = rng.choice([1, 2])
        c["T"] = rng.randint(129, 512 if c["B"] == 1 else 256)
        c["kv_hi"] = _log(rng, 512, 4096)
        c["kv_lo"] = c["kv_hi"] // 2
        return c
    if kind == "topk":
        f32 = rng.random() < 0.4
        V = _log(rng, 8000, 131072)
        if rng.random() < 0.5:
            V = V // 64 * 64
        R = _log(rng, 17, max(17, min(1040, 130000000 // V // (2 if f32 else 1))))
        return dict(kind="topk", R=R, V=V, k=rng.choice([1, 4, 5, 8, 10]), f32=f32)
    if kind == "sample":
        V = _log(rng, 8000, 128256)
        return dict(kind="sample", B=_log(rng, 1, 16), T=rng.randint(8, 64), V=V,
                    temp=rng.choice([0.7, 1.0]))
    return dict(kind="update", B=_log(rng, 1, 64), Hkv=8, D=128, T=rng.randint(8, 96), V=32000,
                k=rng.choice([4, 8]), e_max=rng.choice([512, 2048]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dtype(c):
    return torch.float32 if c["kind"] == "step" else torch.bfloat16


def _lens(c):
    """Committed lengths and live tree sizes of the sequences: the case's own,
    whatever the seed of its values."""
    if c["kind"] != "attn":
        return [c["kv"]], [c["T"]]
    r = random.Random(c["lens"])
    kv = [r.randint(c["kv_lo"], c["kv_hi"]) for _ in range(c["B"])]
    T = c["T"]
    live = [r.randint(max(1, T // 3), T) if c["ragged"] else T for _ in range(c["B"])]
    return kv, live


def _tree(rng, T):
    """Breadth-first forest of T nodes: up to 4, 3, 2, 2, 2, ... children."""
    parent, frontier, d = [], [-1], 0
    while len(parent) < T:
        w = [4, 3, 2][min(d, 2)]
        nxt = []
        for p in frontier:
            for _ in range(w if p < 0 else int(rng.integers(1, w + 1))):
                if len(parent) == T:
                    break
                parent.append(p)
                nxt.append(len(parent) - 1)
        frontier, d = nxt, d + 1
    return np.asarray(parent, np.int32)


def _tokens(rng, parent, V):
    """Token ids, distinct among siblings."""
    tok = np.empty(parent.shape[0], np.int32)
    for p in np.unique(parent):
        kids = np.flatnonzero(parent == p)
        tok[kids] = rng.choice(V, size=kids.size, replace=False)
    return tok


def _trees(c, seed, B):
    rng = np.random.default_rng(seed)
    parent = np.stack([_tree(rng, c["T"]) for _ in range(B)])
    tokens = np.stack([_tokens(rng, p, c["V"]) for p in parent]) if "V" in c else None
    return rng, parent, tokens


def _cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) + 1)


def _i32(*shape):
    return torch.empty(shape, dtype=torch.int32, device=DEV)


def _status():
    return torch.zeros(1, dtype=torch.int32, device=DEV)


def _attn_inputs(c, seed):
    g = _gen(seed)
    dt = _dtype(c)
    kv, live = _lens(c)
    B, T, D = len(kv), c["T"], c["D"]
    page = c.get("page", 0)
    L = max(kv) + T
    L = -(-L // page) * page if page else L
    _, parent, _ = _trees({"T": T}, seed, B)
    s = dict(c=c, T=T, parent=_cu(parent), status=_status(),
             kv_len=torch.tensor(kv, dtype=torch.int32, device=DEV),
             tree_len=torch.tensor(live, dtype=torch.int32, device=DEV)
             if c.get("ragged") else None,
             q=torch.randn((B, T, c["Hq"], D), generator=g, device=DEV, dtype=dt))
    if page:
        n = B * (L // page)
        shape = (n, c["Hkv"], page, D)
        s["table"] = torch.randperm(n, generator=g, device=DEV).to(torch.int32).view(B, L // page)
    else:
        shape = (B, c["Hkv"], L, D)
    s["k"] = torch.randn(shape, generator=g, device=DEV, dtype=dt)
    s["v"] = torch.randn(shape, generator=g, device=DEV, dtype=dt)
    s["ks"] = s["vs"] = None
    if c.get("f8"):
        for n, sc in (("k", "ks"), ("v", "vs")):
            scale = (s[n].abs().amax(dim=(0, 2, 3)).float() / 448.0).contiguous()
            s[n] = (s[n].float() / scale[None, :, None, None]).to(torch.float8_e4m3fn).view(torch.uint8)
            s[sc] = scale
    code = P.PTD_F32 if dt == torch.float32 else P.PTD_BF16
    s["shape"] = P.AttnShape(B, c["Hq"], c["Hkv"], D, L, code, code, 0.0)
    s["ws"] = torch.empty(max(1, P.ptd_tree_attention_workspace_bytes(s["shape"], T)),
                          dtype=torch.uint8, device=DEV)
    s["out"] = torch.empty_like(s["q"])
    if page:
        s["pages"] = P.KVPages(s["k"].data_ptr(), s["v"].data_ptr(), s["table"].data_ptr(), page,
                               L // page, n_pages(s))
    return s


def n_pages(s):
    return s["k"].shape[0]


def _topk_buffers(R, V, k):
    n = P.ptd_topk_workspace_bytes(R, V, k)
    return dict(am=_i32(R), idx=_i32(R, k),
                val=torch.empty((R, k), dtype=torch.float32, device=DEV),
                tws=torch.empty(max(1, n), dtype=torch.uint8, device=DEV))


def _update_buffers(B, T):
    return dict(al=_i32(B), an=_i32(B, T), ot=_i32(B, T + 1), pn=_i32(B, T), tn=_i32(B, T),
                ln=_i32(B))


def _path(rng, parent):
    """A root path of random depth (possibly empty), shallowest first."""
    a = int(rng.integers(-1, parent.shape[0]))
    path = []
    while a >= 0:
        path.append(a)
        a = int(parent[a])
    return path[::-1]


WIDTH = [4, 3, 2, 2, 2, 2]


def prepare(case, seed):
    c = case
    if c["kind"] == "attn" or c["kind"] == "layer":
        return _attn_inputs(c, seed)
    if c["kind"] == "step":
        s = _attn_inputs(c, seed)
        rng, parent, tokens = _trees(c, seed, 1)
        lg = (rng.standard_normal((c["T"] + 1, c["V"])) * LOGIT_STD).astype(np.float32)
        prev = 0
        for a in _path(rng, parent[0]):
            lg[prev, tokens[0, a]] = 16.0
            prev = a + 1
        s.update(parent=_cu(parent), tokens=_cu(tokens), logits=_cu(lg),
                 **_topk_buffers(c["T"] + 1, c["V"], c["k"]), **_update_buffers(1, c["T"]))
        return s
    if c["kind"] == "topk":
        lg = torch.randn((c["R"], c["V"]), generator=_gen(seed), device=DEV) * LOGIT_STD
        return dict(c=c, logits=lg if c["f32"] else lg.to(torch.bfloat16),
                    **_topk_buffers(c["R"], c["V"], c["k"]))
    if c["kind"] == "sample":
        B, T, V = c["B"], c["T"], c["V"]
        g = _gen(seed)
        rng, parent, tokens = _trees(c, seed, B)
        lg = torch.randn((B * (T + 1), V), generator=g, device=DEV) * LOGIT_STD
        # draft tokens are likely ones: about 0.1 to 0.6 of their row's mass
        rows = _cu((np.arange(B)[:, None] * (T + 1) + parent + 1).astype(np.int64))
        top = c["temp"] * (math.log(V) + 0.5 * (LOGIT_STD / c["temp"]) ** 2)
        spike = top + c["temp"] * (torch.rand((B, T), generator=g, device=DEV) * 2.5 - 2.0)
        lg[rows.view(-1), _cu(tokens.astype(np.int64)).view(-1)] = spike.view(-1)
        return dict(c=c, logits=lg.to(torch.bfloat16), parent=_cu(parent), tokens=_cu(tokens),
                    u_node=torch.rand((B, T), generator=g, dtype=torch.float64, device=DEV),
                    u_bonus=torch.rand((B, T + 1), generator=g, dtype=torch.float64, device=DEV),
                    al=_i32(B), an=_i32(B, T), ot=_i32(B, T + 1), status=_status(),
                    ws=torch.empty(P.ptd_verify_sample_workspace_bytes(B, T, V),
                                   dtype=torch.uint8, device=DEV))
    # update
    B, T, V, k = c["B"], c["T"], c["V"], c["k"]
    rng, parent, tokens = _trees(c, seed, B)
    argmax = rng.integers(0, V, (B, T + 1)).astype(np.int32)
    topk = rng.integers(0, V, (B, T + 1, k)).astype(np.int32)
    last = np.empty(B, np.int32)
    for b in range(B):
        prev = 0
        for a in _path(rng, parent[b]):
            argmax[b, prev] = tokens[b, a]
            prev = a + 1
        # the bonus token: one that the drafts have seen, so the pool knows it
        argmax[b, prev] = last[b] = tokens[b, int(rng.integers(0, T))]
    topk[:, :, 0] = argmax
    kv = rng.integers(128, 512, B).astype(np.int32)
    g = _gen(seed)
    L = int(kv.max()) + T
    s = dict(c=c, parent=_cu(parent), tokens=_cu(tokens), argmax=_cu(argmax), topk=_cu(topk),
             last=_cu(last), kv_len=_cu(kv), kv_next=_i32(B), status=_status(),
             k=torch.randn((B, c["Hkv"], L, c["D"]), generator=g, device=DEV, dtype=torch.bfloat16),
             v=torch.randn((B, c["Hkv"], L, c["D"]), generator=g, device=DEV, dtype=torch.bfloat16),
             shape=P.AttnShape(B, c["Hkv"], c["Hkv"], c["D"], L, P.PTD_BF16, P.PTD_BF16, 0.0),
             pool=P.Pool(B, c["e_max"], T + 1, device=DEV), **_update_buffers(B, T))
    s.update(sp=_i32(B, T), st=_i32(B, T), sl=_i32(B), rp=_i32(B, T), rt=_i32(B, T), rl=_i32(B))
    # earlier steps' drafts are in the pool
    for _ in range(3):
        s["pool"].merge(s["parent"], _cu(np.stack([_tokens(rng, p, V) for p in parent])))
    s["pool"].merge(s["parent"], s["tokens"])
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _attention(s):
    T, ws = s["T"], s["ws"]
    c = s["c"]
    if c.get("page"):
        if c["f8"]:
            P.ptd_tree_attention_paged_fp8kv(s["q"], s["pages"], s["ks"], s["vs"], s["kv_len"],
                                             s["tree_len"], s["parent"], T, s["out"], s["shape"],
                                             ws, ws.numel(), s["status"])
        else:
            P.ptd_tree_attention_paged(s["q"], s["pages"], s["kv_len"], s["tree_len"],
                                       s["parent"], T, s["out"], s["shape"], None, ws, ws.numel(),
                                       s["status"])
    elif s["tree_len"] is not None:
        P.ptd_tree_attention_ragged(s["q"], s["k"], s["v"], s["kv_len"], s["tree_len"],
                                    s["parent"], T, s["out"], s["shape"], None, ws, ws.numel(),
                                    s["status"])
    else:
        P.ptd_tree_attention(s["q"], s["k"], s["v"], s["kv_len"], s["parent"], T, s["out"],
                             s["shape"], None, ws, ws.numel(), s["status"])


def _topk(s, R, V, k, code):
    P.ptd_topk_argmax(s["logits"], code, R, V, V, k, s["am"], s["idx"], s["val"], s["tws"],
                      s["tws"].numel())


def _verify_expand(s, am, idx, B, T, k):
    P.ptd_verify_expand(am, s["tokens"], s["parent"], None, B, T, idx, k, WIDTH, len(WIDTH), T,
                        s["al"], s["an"], s["ot"], s["pn"], s["tn"], s["ln"], s["status"])


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "attn":
        _attention(s)
        return dict(out=s["out"], status=s["status"])
    if c["kind"] == "layer":
        P.ptd_tree_rope(s["q"], s["k"], s["kv_len"], s["parent"], s["T"], s["shape"],
                        dev_status=s["status"])
        _attention(s)
        return dict(out=s["out"], q=s["q"], k=s["k"], status=s["status"])
    if c["kind"] == "step":
        T = c["T"]
        _attention(s)
        _topk(s, T + 1, c["V"], c["k"], P.PTD_F32)
        _verify_expand(s, s["am"], s["idx"], 1, T, c["k"])
        return {n: s[n] for n in ("out", "am", "idx", "val", "al", "an", "ot", "pn", "tn", "ln",
                                  "status")}
    if c["kind"] == "topk":
        _topk(s, c["R"], c["V"], c["k"], P.PTD_F32 if c["f32"] else P.PTD_BF16)
        return {n: s[n] for n in ("am", "idx", "val")}
    if c["kind"] == "sample":
        P.ptd_verify_sample(s["logits"], P.PTD_BF16, c["V"], c["V"], s["tokens"], s["parent"],
                            None, c["B"], c["T"], c["temp"], s["u_node"], s["u_bonus"], s["al"],
                            s["an"], s["ot"], s["ws"], s["ws"].numel(), s["status"])
        return {n: s[n] for n in ("al", "an", "ot", "status")}
    B, T = c["B"], c["T"]
    _verify_expand(s, s["argmax"], s["topk"], B, T, c["k"])
    P.ptd_kv_commit(s["k"], s["v"], s["kv_len"], s["al"], s["an"], T, s["shape"], s["kv_next"],
                    s["status"])
    P.ptd_step_prune(s["pn"], s["tn"], s["ln"], B, T, len(WIDTH) - 1, T, s["sp"], s["st"],
                     s["sl"], s["status"])
    pool = s["pool"]
    P.ptd_pool_merge(pool.buf, pool.nbytes, B, pool.e_max, pool.n_cap, s["sp"], s["st"], s["sl"],
                     T, s["status"])
    P.ptd_pool_retrieve(pool.buf, pool.nbytes, B, pool.e_max, pool.n_cap, s["last"], T, s["rp"],
                        s["rt"], s["rl"])
    return {n: s[n] for n in ("al", "an", "ot", "pn", "tn", "ln", "kv_next", "k", "v", "sp", "st",
                              "sl", "rp", "rt", "rl", "status")}


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far correct results lie apart
# ---------------------------------------------------------------------------
def work(case):
    c = case
    if c["kind"] == "topk":
        return {"bytes": c["R"] * (c["V"] * (4 if c["f32"] else 2) + 4 + 8 * c["k"]),
                "flops": c["R"] * c["V"]}
    if c["kind"] == "sample":
        n = c["B"] * (c["T"] + 1)
        return {"bytes": n * c["V"] * 2 + n * 40, "flops": 3 * n * c["V"]}
    if c["kind"] == "update":
        # trees and their successors, the draft's sub-trees in the pool, a few moved rows
        n = c["B"] * c["T"]
        return {"bytes": n * (12 + 4 * c["k"] + 40) + c["B"] * 2 * 2 * 3 * c["Hkv"] * c["D"] * 2,
                "flops": 0}
    kv, live = _lens(c)
    es = 4 if c["kind"] == "step" else 2
    kes = 1 if c.get("f8") else es
    keys, nodes = sum(kv) + sum(live), sum(live)
    b = 2 * keys * c["Hkv"] * c["D"] * kes + 2 * nodes * c["Hq"] * c["D"] * es
    f = 4 * c["Hq"] * c["D"] * sum(n * k for n, k in zip(live, kv))
    if c["kind"] == "layer":  # the embedding turns q and the tree's keys in place
        b += nodes * (c["Hq"] + c["Hkv"]) * c["D"] * es
    if c["kind"] == "step":
        b += (c["T"] + 1) * c["V"] * es
    return {"bytes": b, "flops": f}


def tolerance(case):
    c = case
    if c["kind"] in ("topk", "sample", "update"):
        return "exact"
    if c["kind"] == "step":  # fp32 throughout
        return {"rel": 2e-6}
    return {"rel": 1e-2}  # bf16 outputs (2.4e-3 from 64 bits); the softmax weights are bf16 too


def exact(case, seed):
    c = case
    if c["kind"] in ("sample", "update"):
        return None
    s = prepare(case, seed)
    if c["kind"] == "topk":
        return dict(am=None, idx=None, val=torch.topk(s["logits"].double(), c["k"], dim=1).values)
    kv, live = _lens(c)
    B, T, Hq, D = s["q"].shape
    Hkv, G = c["Hkv"], c["Hq"] // c["Hkv"]
    q, parent = s["q"].double(), s["parent"].cpu().numpy()
    anc = np.zeros((B, T, T), bool)
    for b in range(B):
        for i in range(T):
            if parent[b, i] >= 0:
                anc[b, i] = anc[b, parent[b, i]]
            anc[b, i, i] = True
    kc = s["k"].double() if c["kind"] == "layer" else None
    if c["kind"] == "layer":
        pos = torch.as_tensor(kv[0] + anc[0].sum(1) - 1, dtype=torch.float64, device=DEV)
        inv = 10000.0 ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device=DEV) / D)
        cos, sin = torch.cos(pos[:, None] * inv), torch.sin(pos[:, None] * inv)

        def turn(x):  # [T][heads][D], pairs (p, p + D/2)
            a, b2 = x[..., :D // 2], x[..., D // 2:]
            cs, sn = cos[:, None], sin[:, None]
            return torch.cat((a * cs - b2 * sn, a * sn + b2 * cs), -1)

        q[0] = turn(q[0])
        rows = slice(kv[0], kv[0] + T)
        kc[0, :, rows] = turn(kc[0, :, rows].transpose(0, 1)).transpose(0, 1)
    out = torch.zeros((B, T, Hq, D), dtype=torch.float64, device=DEV)
    for b in range(B):
        N = kv[b] + live[b]

        def rows_of(x, scale):
            if c.get("page"):
                t = s["table"][b].long()
                r = x[t].transpose(0, 1).reshape(Hkv, -1, D)[:, :N]
            else:
                r = x[b, :, :N]
            if c.get("f8"):
                return r.contiguous().view(torch.float8_e4m3fn).double() * scale.double()[:, None, None]
            return r.double()

        K = kc[b, :, :N] if kc is not None else rows_of(s["k"], s["ks"])
        Vv = rows_of(s["v"], s["vs"])
        vis = torch.ones((live[b], N), dtype=torch.bool, device=DEV)
        vis[:, kv[b]:] = _cu(anc[b, :live[b], :live[b]])
        for g in range(Hkv):
            qg = q[b, :live[b], g * G:(g + 1) * G].reshape(-1, D)
            x = (qg @ K[g].t().contiguous()) / math.sqrt(D)
            x = x.view(live[b], G, N).masked_fill(~vis[:, None], -math.inf).view(-1, N)
            out[b, :live[b], g * G:(g + 1) * G] = (torch.softmax(x, 1) @ Vv[g]).view(live[b], G, D)
    if c["kind"] == "attn":
        return dict(out=out, status=None)
    if c["kind"] == "layer":
        return dict(out=out, q=q, k=kc, status=None)
    return dict(out=out, val=torch.topk(s["logits"].double(), c["k"], dim=1).values,
                **{n: None for n in ("am", "idx", "al", "an", "ot", "pn", "tn", "ln", "status")})
