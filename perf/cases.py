"""Performance cases of libcas: one attention layer's calls as programs make them.

Every case is one pass through the public entry points of the Python binding:

* ``train``    prefix_attn_fwd and prefix_attn_bwd on one batch (fixed rows or
               packed samples): the layer's share of a training step. Returns
               O, LSE, dQ, the self dK/dV and every cartridge's dK/dV.
* ``prefill``  prefix_attn_fwd (or prefix_attn_fwd_noalloc) alone: prompts over
               retrieved cartridges. Returns O and LSE.
* ``decode``   paged_decode_fwd: the new tokens of running requests over pages
               of retrieved cartridges and of their own. Returns O and LSE.
* ``adam``     cartridge_adam: the optimizer step of the active cartridges.
               Returns the parameters and the moments it wrote.

The sizes of a case are plain values; what they leave open (ragged lengths,
which cartridges a row selects) comes from ``shape_seed``, so two seeds of one
case differ in their data and not in their work. Tensors are seeded Gaussians
with the workloads' distributions (queries, self K/V and dO of unit variance,
cartridge K/V of standard deviation 0.5). Cartridges are views of pools, as a
program with a fixed budget of slots holds them.
"""
import math
import random

import torch

import paper_2606_04557_amd as cas

DEV = "cuda"


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _train(name=None, **kw):
    c = dict(kind="train", dtype="bf16", batch=1, q_len=0, tokens=0, q_lo=0, q_hi=0, kv_heads=8, group=4, head_dim=128,
             carts=1, pool=0, len_lo=1024, len_hi=1024, len_step=1, layout="tok", shape_seed=1)
    c.update(kw)
    return dict(name=name, **c) if name else c


def _prefill(name=None, **kw):
    c = dict(kind="prefill", dtype="bf16", batch=1, q_len=64, tokens=0, q_lo=0, q_hi=0, kv_heads=8, group=4, head_dim=128,
             carts=4, pool=0, len_lo=1024, len_hi=1024, len_step=1, layout="tok", noalloc=False, shape_seed=1)
    c.update(kw)
    return dict(name=name, **c) if name else c


def _decode(name=None, **kw):
    c = dict(kind="decode", batch=1, new=1, kv_heads=8, group=4, head_dim=128, page=16, carts=4, pool=8, cart_len=1024,
             own_lo=65, own_hi=65, shape_seed=1)
    c.update(kw)
    return dict(name=name, **c) if name else c


def _adam(name=None, **kw):
    c = dict(kind="adam", carts=20, len_lo=256, len_hi=2048, len_step=16, kv_heads=8, head_dim=128, step=7, frozen=1,
             layout="tok", shape_seed=1)
    c.update(kw)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # The headline training shape: a long prefix of 16 cartridges per row.
        _train("train_16x2k", batch=2, q_len=2048, carts=16, len_lo=2048, len_hi=2048),
        # The common training shape: a target and three distractors per row.
        _train("train_4x1k", batch=4, q_len=1024, carts=4),
        # One long ragged prefix (64 cartridges in several storage layouts), few queries: the key axis is split.
        _train("train_ragged64", batch=1, q_len=512, carts=64, len_lo=256, len_hi=4096, layout="mixed", shape_seed=4),
        # The packed layout: samples of different lengths in 8,192 tokens over a shared pool of 20 cartridges.
        _train("train_packed8k", batch=8, tokens=8192, q_lo=256, q_hi=2048, carts=11, pool=20, len_lo=256, len_hi=2048,
               len_step=16, shape_seed=6),
        # A small model's layer with odd sizes: head_dim 64, three heads per group, lengths off every tile edge.
        _train("train_odd_d64", batch=3, q_len=141, kv_heads=4, group=3, head_dim=64, carts=3, len_lo=129, len_hi=500,
               shape_seed=2),
        # fp32, the precision in which a port of a model is checked, at its smallest: latency.
        _train("train_fp32_small", dtype="fp32", q_len=64, kv_heads=2, group=2, head_dim=64, carts=2, len_lo=128,
               len_hi=128),
        # A serving batch's prompts, each over 4 of 256 retrieved cartridges.
        _prefill("prefill_64req", batch=64, q_len=64, pool=256, shape_seed=5),
        # One request's prompt over four cartridges of ragged length, without allocation.
        _prefill("prefill_one_noalloc", batch=1, q_len=137, len_lo=900, len_hi=1500, noalloc=True, shape_seed=3),
        # A decode step of a serving batch, cartridge pages shared between requests.
        _decode("decode_64req", batch=64, pool=256, shape_seed=5),
        # A decode step of a single request: latency.
        _decode("decode_one", batch=1, pool=8, own_lo=211, own_hi=211, shape_seed=3),
        # Several new tokens per request (drafted tokens to verify, or a short user turn).
        _decode("decode_16req_8new", batch=16, new=8, pool=64, own_lo=8, own_hi=300, shape_seed=7),
        # The optimizer step of the whole GPU pool of 20 cartridges.
        _adam("adam_pool20", shape_seed=6),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["train", "train", "packed", "fp32", "prefill", "prefill", "decode", "decode", "adam"])
    seed = rng.randrange(1, 1 << 20)
    if kind in ("train", "fp32", "packed"):
        while True:
            fp32 = kind == "fp32"
            d = rng.choice([64, 128, 128])
            kvh, g = rng.choice([2, 4, 8, 8]), rng.choice([1, 2, 3, 4, 4, 8])
            lo = _logint(rng, 64, 512 if fp32 else 2048)
            c = _train(dtype="fp32" if fp32 else "bf16", batch=rng.randint(1, 4), q_len=_logint(rng, 32, 512 if fp32 else 2048),
                       kv_heads=kvh, group=g, head_dim=d, carts=_logint(rng, 1, 4 if fp32 else 24), len_lo=lo,
                       len_hi=_logint(rng, lo, 512 if fp32 else 4096), layout=rng.choice(["tok", "mixed"]), shape_seed=seed)
            if kind == "packed":
                c["tokens"], c["q_len"], c["batch"] = _logint(rng, 512, 8192), 0, rng.randint(2, 8)
                c["q_lo"], c["q_hi"] = 32, 2048
                c["carts"], c["pool"] = rng.randint(1, 11), 20
                c["len_lo"], c["len_hi"], c["len_step"] = 256, rng.choice([512, 1024, 2048]), 16
            flops = work(c)["flops"]
            if flops <= (1e11 if fp32 else 5e12) and _segment_bytes(c) <= 2e9:
                return c
    if kind == "prefill":
        b = _logint(rng, 1, 64)
        lo = _logint(rng, 256, 2048)
        k = rng.randint(1, 8)
        noalloc = b <= 8 and rng.random() < 0.4
        return _prefill(batch=b, q_len=_logint(rng, 16, max(32, 4096 // b)), kv_heads=rng.choice([4, 8, 8]),
                        group=rng.choice([2, 4, 4, 8]), head_dim=rng.choice([64, 128, 128]), carts=k,
                        pool=rng.choice([16, 64, 128]), len_lo=lo, len_hi=min(2048, lo + rng.randint(0, 300)), noalloc=noalloc,
                        shape_seed=seed)
    if kind == "decode":
        return _decode(batch=_logint(rng, 1, 64), new=rng.choice([1, 1, 1, 2, 4, 5, 8]), kv_heads=rng.choice([4, 8, 8]),
                       group=rng.choice([2, 4, 4, 5, 8]), head_dim=rng.choice([64, 128, 128]), page=rng.choice([16, 16, 32, 64]),
                       carts=rng.randint(1, 8), pool=rng.choice([16, 64, 128]), cart_len=128 * _logint(rng, 2, 12), own_lo=8,
                       own_hi=rng.choice([64, 300, 1000]), shape_seed=seed)
    return _adam(carts=rng.randint(1, 20), len_lo=_logint(rng, 64, 512), len_hi=_logint(rng, 512, 2048),
                 len_step=rng.choice([1, 16]), kv_heads=rng.choice([4, 8, 8]), head_dim=rng.choice([64, 128, 128]),
                 step=rng.randrange(0, 40), frozen=rng.choice([0, 1]), layout=rng.choice(["tok", "mixed"]), shape_seed=seed)


# ---------------------------------------------------------------------------
# Shapes (from the case alone)
# ---------------------------------------------------------------------------
def _shape(c):
    """(row lengths, cartridge lengths, per row cartridge ids, per cartridge layout)."""
    r = random.Random(c["shape_seed"])
    B, k = c["batch"], c["carts"]
    n = c["pool"] if c["pool"] else B * k

    def length():
        return max(c["len_lo"], r.randint(c["len_lo"], c["len_hi"]) // c["len_step"] * c["len_step"])

    lens = [length() for _ in range(n)]
    if c["tokens"]:
        # Packed samples: lengths drawn, then scaled to fill the token axis; one in four rows sees distractors.
        q = [r.randint(c["q_lo"], c["q_hi"]) for _ in range(B)]
        q = [max(1, x * c["tokens"] // sum(q)) for x in q]
        q[-1] += c["tokens"] - sum(q)
        rows = [r.sample(range(n), 1 if r.random() < 0.75 else r.randint(1, k)) for _ in range(B)]
    else:
        q = [c["q_len"]] * B
        rows = [r.sample(range(n), min(k, n)) for _ in range(B)] if c["pool"] else [list(range(b * k, b * k + k)) for b in range(B)]
    lay = [r.choice(["tok", "tok", "padded", "head"]) if c["layout"] == "mixed" else "tok" for _ in range(n)]
    return q, lens, rows, lay


def _segment_bytes(c):
    _, lens, rows, _ = _shape(c)
    used = {i for row in rows for i in row}
    return sum(lens[i] for i in used) * c["kv_heads"] * c["head_dim"] * (2 if c.get("dtype", "bf16") == "bf16" else 4)


def _decode_shape(c):
    """(new tokens, key counts, page lists, pages of the pool) of the requests."""
    r = random.Random(c["shape_seed"])
    P, cp = c["page"], c["cart_len"] // c["page"]
    nxt = c["pool"] * cp
    q, kv, pages = [], [], []
    for _ in range(c["batch"]):
        ids = [i * cp + j for i in r.sample(range(c["pool"]), min(c["carts"], c["pool"])) for j in range(cp)]
        own = max(c["new"], r.randint(c["own_lo"], c["own_hi"]))
        op = -(-own // P)
        pages.append(ids + list(range(nxt, nxt + op)))
        nxt += op
        kv.append(len(ids) * P + own)
        q.append(c["new"])
    return q, kv, pages, nxt


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _randn(gen, shape, std, dtype):
    return (torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32) * std).to(dtype)


def _slot_elems(L, H, D, lay):
    return L * (H * D + 64) if lay == "padded" else L * H * D


def _view(flat, at, L, H, D, lay):
    """The [L, H, D] view of a cartridge in its slot of a flat pool."""
    x = flat[at: at + _slot_elems(L, H, D, lay)]
    if lay == "padded":
        return x.view(L, H * D + 64)[:, : H * D].view(L, H, D)
    if lay == "head":
        return x.view(H, L, D).permute(1, 0, 2)
    return x.view(L, H, D)


def _slots(lens, lay, H, D):
    at, off = [], 0
    for L, y in zip(lens, lay):
        at.append(off)
        off += -(-_slot_elems(L, H, D, y) // 64) * 64
    return at, off


def _attn_inputs(c, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    q_lens, lens, rows, lay = _shape(c)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    H, g, D = c["kv_heads"], c["group"], c["head_dim"]
    packed = bool(c["tokens"])
    lead = (sum(q_lens),) if packed else (c["batch"], c["q_len"])
    at, total = _slots(lens, lay, H, D)
    t = {"q": _randn(gen, lead + (H * g, D), 1.0, dt), "k_self": _randn(gen, lead + (H, D), 1.0, dt),
         "v_self": _randn(gen, lead + (H, D), 1.0, dt), "k_pool": _randn(gen, (total,), 0.5, dt),
         "v_pool": _randn(gen, (total,), 0.5, dt)}
    if c["kind"] == "train":
        t["d_o"] = _randn(gen, lead + (H * g, D), 1.0, dt)
    offs = [0]
    for n in q_lens:
        offs.append(offs[-1] + n)
    return t, q_lens, lens, rows, lay, at, total, offs if packed else None


def _decode_inputs(c, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    q_counts, kv, pages, npages = _decode_shape(c)
    H, g, D, P = c["kv_heads"], c["group"], c["head_dim"], c["page"]
    k = _randn(gen, (npages, P, H, D), 0.5, torch.bfloat16)
    v = _randn(gen, (npages, P, H, D), 0.5, torch.bfloat16)
    q = _randn(gen, (sum(q_counts), H * g, D), 1.0, torch.bfloat16)
    return q, k, v, q_counts, kv, pages, npages


def _adam_inputs(c, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    r = random.Random(c["shape_seed"])
    lens = [max(c["len_lo"], r.randint(c["len_lo"], max(c["len_lo"], c["len_hi"])) // c["len_step"] * c["len_step"])
            for _ in range(c["carts"])]
    lay = [r.choice(["tok", "tok", "padded", "head"]) if c["layout"] == "mixed" else "tok" for _ in lens]
    steps = [max(0, c["step"] - r.randint(0, 10)) for _ in lens]
    H, D = c["kv_heads"], c["head_dim"]
    at, total = _slots(lens, lay, H, D)
    m_at, m_total = _slots(lens, ["tok"] * len(lens), H, D)
    t = {n: _randn(gen, (total,), std, torch.bfloat16) for n, std in (("k", 0.5), ("v", 0.5), ("dk", 0.02), ("dv", 0.02))}
    for n in ("m1_k", "m1_v"):
        t[n] = _randn(gen, (m_total,), 0.01, torch.float32)
    for n in ("m2_k", "m2_v"):
        t[n] = _randn(gen, (m_total,), 0.02, torch.float32).square_()
    return t, lens, lay, steps, at, m_at


def prepare(case, seed):
    c = case
    scale = 1.0 / math.sqrt(c["head_dim"])
    if c["kind"] in ("train", "prefill"):
        t, q_lens, lens, rows, lay, at, total, offs = _attn_inputs(c, seed)
        H, g, D = c["kv_heads"], c["group"], c["head_dim"]
        train = c["kind"] == "train"
        if train:
            # Zeroed: the padding between rows, and cartridges that no row selects, are not written.
            t["dk_pool"], t["dv_pool"] = torch.zeros_like(t["k_pool"]), torch.zeros_like(t["v_pool"])
            t["dq"], t["dk_self"], t["dv_self"] = (torch.empty_like(t[n]) for n in ("q", "k_self", "v_self"))
        segs = [cas.Segment(*(_view(t[n], at[i], lens[i], H, D, lay[i])
                              for n in (("k_pool", "v_pool", "dk_pool", "dv_pool") if train else ("k_pool", "v_pool"))))
                for i in range(len(lens))]
        table = [[segs[i] for i in row] for row in rows]
        prob = cas.Problem.from_tensors(t["q"], table, H, g, scale, offs)
        ws = cas.workspace_size(prob, False)
        if train:
            ws = max(ws, cas.workspace_size(prob, True))
        t["o"] = torch.empty_like(t["q"])
        T = sum(q_lens)
        t["lse"] = torch.empty((H * g, T) if offs else (c["batch"], H * g, c["q_len"]), dtype=torch.float32, device=DEV)
        return dict(c=c, t=t, rows=table, scale=scale, offs=offs, ws=torch.empty(max(ws, 1), dtype=torch.uint8, device=DEV))
    if c["kind"] == "decode":
        q, k, v, q_counts, kv, pages, npages = _decode_inputs(c, seed)
        prob = cas.DecodeProblem(q_counts, kv, pages, npages, c["page"], c["kv_heads"], c["group"], c["head_dim"], scale)
        return dict(c=c, q=q, k=k, v=v, q_counts=q_counts, kv=kv, pages=pages, scale=scale, prob=prob, o=torch.empty_like(q),
                    lse=torch.empty((q.shape[1], q.shape[0]), dtype=torch.float32, device=DEV))
    t, lens, lay, steps, at, m_at = _adam_inputs(c, seed)
    H, D = c["kv_heads"], c["head_dim"]
    carts = [cas.AdamCartridge(*(_view(t[n], at[i], lens[i], H, D, lay[i]) for n in ("k", "v", "dk", "dv")),
                               *(_view(t[n], m_at[i], lens[i], H, D, "tok") for n in ("m1_k", "m2_k", "m1_v", "m2_v")),
                               step=steps[i], frozen_tokens=c["frozen"]) for i in range(len(lens))]
    return dict(c=c, t=t, carts=carts)


def run(state):
    c = state["c"]
    if c["kind"] == "adam":
        cas.cartridge_adam(state["carts"], 1e-3)
        t = state["t"]
        return {n: t[n] for n in ("k", "v", "m1_k", "m2_k", "m1_v", "m2_v")}
    if c["kind"] == "decode":
        s = state
        o, lse = cas.paged_decode_fwd(s["q"], s["k"], s["v"], s["q_counts"], s["kv"], s["pages"], c["kv_heads"], c["group"],
                                      s["scale"], o=s["o"], lse=s["lse"], problem=s["prob"])
        return {"o": o, "lse": lse}
    t, H, g = state["t"], c["kv_heads"], c["group"]
    if c["kind"] == "prefill" and c["noalloc"]:
        cas.prefix_attn_fwd_noalloc(t["q"], t["k_self"], t["v_self"], state["rows"], H, g, state["scale"], t["o"], t["lse"],
                                    q_offsets=state["offs"])
        return {"o": t["o"], "lse": t["lse"]}
    o, lse = cas.prefix_attn_fwd(t["q"], t["k_self"], t["v_self"], state["rows"], H, g, state["scale"], o=t["o"], lse=t["lse"],
                                 workspace=state["ws"], q_offsets=state["offs"])
    if c["kind"] == "prefill":
        return {"o": o, "lse": lse}
    dq, dks, dvs = cas.prefix_attn_bwd(t["q"], t["k_self"], t["v_self"], state["rows"], H, g, state["scale"], o, lse, t["d_o"],
                                       dq=t["dq"], dk_self=t["dk_self"], dv_self=t["dv_self"], workspace=state["ws"],
                                       q_offsets=state["offs"])
    return {"o": o, "lse": lse, "dq": dq, "dk_self": dks, "dv_self": dvs, "dk": t["dk_pool"], "dv": t["dv_pool"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how close its outputs have to be
# ---------------------------------------------------------------------------
def work(case):
    c = case
    if c["kind"] == "adam":
        r = random.Random(c["shape_seed"])
        lens = [max(c["len_lo"], r.randint(c["len_lo"], max(c["len_lo"], c["len_hi"])) // c["len_step"] * c["len_step"])
                for _ in range(c["carts"])]
        n = sum(max(0, L - c["frozen"]) for L in lens) * c["kv_heads"] * c["head_dim"] * 2
        # bf16 parameter and gradient read, parameter written; two fp32 moments read and written.
        return {"bytes": 22 * n, "flops": 14 * n}
    H, g, D = c["kv_heads"], c["group"], c["head_dim"]
    if c["kind"] == "decode":
        q, kv, pages, _ = _decode_shape(c)
        used = len({p for pl in pages for p in pl})   # a page shared by requests is read once
        pairs = sum(sum(L - n + i + 1 for i in range(n)) for n, L in zip(q, kv)) * H * g
        return {"bytes": 2 * used * c["page"] * H * D * 2 + sum(q) * H * g * (4 * D + 4), "flops": 4 * D * pairs}
    es = 2 if c["dtype"] == "bf16" else 4
    q_lens, lens, rows, _ = _shape(c)
    T = sum(q_lens)
    used = {i for row in rows for i in row}
    kv = 2 * (sum(lens[i] for i in used) + T) * H * D * es            # K and V, cartridges and self
    qb, stat = T * H * g * D * es, T * H * g * 4
    pairs = sum(n * sum(lens[i] for i in row) + n * (n + 1) // 2 for n, row in zip(q_lens, rows)) * H * g
    if c["kind"] == "prefill":
        return {"bytes": kv + 2 * qb + stat, "flops": 4 * D * pairs}
    # Forward: Q, K, V in, O, LSE out. Backward: those and dO in, dQ, dK, dV out.
    return {"bytes": (kv + 2 * qb + stat) + (2 * kv + 4 * qb + stat), "flops": 12 * D * pairs}


def tolerance(case):
    if case["kind"] == "adam":
        return "exact"   # every operation rounds once, in the documented order
    if case.get("dtype") == "fp32":
        return {"rel": 4e-6, "max": 1e-4}
    return {"rel": 1e-2, "max": 2e-1}


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _exact_attn(c, seed):
    t, q_lens, lens, rows, lay, at, total, offs = _attn_inputs(c, seed)
    H, g, D = c["kv_heads"], c["group"], c["head_dim"]
    scale, train = 1.0 / math.sqrt(D), c["kind"] == "train"
    T = sum(q_lens)
    f = torch.float64
    q = t["q"].reshape(T, H, g, D).to(f)
    ks, vs = t["k_self"].reshape(T, H, D).to(f), t["v_self"].reshape(T, H, D).to(f)
    o = torch.zeros(T, H, g, D, dtype=f, device=DEV)
    lse = torch.zeros(H * g, T, dtype=f, device=DEV)
    if train:
        do = t["d_o"].reshape(T, H, g, D).to(f)
        dq, dks, dvs = torch.zeros_like(q), torch.zeros_like(ks), torch.zeros_like(vs)
        dk_pool, dv_pool = (torch.zeros(total, dtype=f, device=DEV) for _ in range(2))
    tok = 0
    for n, row in zip(q_lens, rows):
        P = sum(lens[i] for i in row)
        mask = torch.zeros(n, 1, P + n, dtype=torch.bool, device=DEV)
        mask[:, 0, P:] = torch.ones(n, n, dtype=torch.bool, device=DEV).triu(1)
        mask = mask.expand(n, g, P + n).reshape(n * g, P + n)
        sl = slice(tok, tok + n)
        for h in range(H):
            K = torch.cat([_view(t["k_pool"], at[i], lens[i], H, D, lay[i])[:, h].to(f) for i in row] + [ks[sl, h]])
            V = torch.cat([_view(t["v_pool"], at[i], lens[i], H, D, lay[i])[:, h].to(f) for i in row] + [vs[sl, h]])
            Q = q[sl, h].reshape(n * g, D)
            S = (Q @ K.T).mul_(scale).masked_fill_(mask, -math.inf)
            L = torch.logsumexp(S, 1)
            Pm = S.sub_(L[:, None]).exp_()
            O = Pm @ V
            o[sl, h] = O.view(n, g, D)
            lse[h * g:(h + 1) * g, sl] = L.view(n, g).T
            if train:
                dO = do[sl, h].reshape(n * g, D)
                dV = Pm.T @ dO
                dS = (dO @ V.T).sub_((dO * O).sum(1, keepdim=True)).mul_(Pm)
                dq[sl, h] = (dS @ K).mul_(scale).view(n, g, D)
                dK = (dS.T @ Q).mul_(scale)
                x = 0
                for i in row:
                    _view(dk_pool, at[i], lens[i], H, D, lay[i])[:, h] += dK[x: x + lens[i]]
                    _view(dv_pool, at[i], lens[i], H, D, lay[i])[:, h] += dV[x: x + lens[i]]
                    x += lens[i]
                dks[sl, h] += dK[x:]
                dvs[sl, h] += dV[x:]
        tok += n
    if not offs:
        lse = lse.view(H * g, c["batch"], c["q_len"]).permute(1, 0, 2)
    out = {"o": o.reshape(t["q"].shape), "lse": lse.contiguous()}
    if train:
        out.update(dq=dq.reshape(t["q"].shape), dk_self=dks.reshape(t["k_self"].shape), dv_self=dvs.reshape(t["k_self"].shape),
                   dk=dk_pool, dv=dv_pool)
    return out


def _exact_decode(c, seed):
    q, k, v, q_counts, kv, pages, _ = _decode_inputs(c, seed)
    H, g, D = c["kv_heads"], c["group"], c["head_dim"]
    f = torch.float64
    o = torch.zeros(q.shape, dtype=f, device=DEV)
    lse = torch.zeros(q.shape[1], q.shape[0], dtype=f, device=DEV)
    tok = 0
    for n, L, pl in zip(q_counts, kv, pages):
        ids = torch.tensor(pl, device=DEV)
        K = k[ids].reshape(-1, H, D)[:L].to(f)
        V = v[ids].reshape(-1, H, D)[:L].to(f)
        last = torch.arange(L - n, L, device=DEV).repeat_interleave(g)
        hide = torch.arange(L, device=DEV)[None, :] > last[:, None]
        for h in range(H):
            Q = q[tok: tok + n, h * g:(h + 1) * g].to(f).reshape(n * g, D)
            S = (Q @ K[:, h].T).mul_(1.0 / math.sqrt(D)).masked_fill_(hide, -math.inf)
            Z = torch.logsumexp(S, 1)
            o[tok: tok + n, h * g:(h + 1) * g] = (S.sub_(Z[:, None]).exp_() @ V[:, h]).view(n, g, D)
            lse[h * g:(h + 1) * g, tok: tok + n] = Z.view(n, g).T
        tok += n
    return {"o": o, "lse": lse}


def _exact_adam(c, seed):
    t, lens, lay, steps, at, m_at = _adam_inputs(c, seed)
    H, D, b1, b2, eps, lr, W, N = c["kv_heads"], c["head_dim"], 0.9, 0.999, 1e-8, 1e-3, 20, 4
    out = {n: t[n].to(torch.float64) for n in ("k", "v", "m1_k", "m2_k", "m1_v", "m2_v")}
    for i, (L, y, s) in enumerate(zip(lens, lay, steps)):
        rate = lr if s >= W else lr * max(1, -(-N * s // W)) / N
        for n in ("k", "v"):
            cut = slice(c["frozen"], L)
            x = _view(out[n], at[i], L, H, D, y)[cut]
            gr = _view(t["d" + n], at[i], L, H, D, y)[cut].to(torch.float64)
            m1, m2 = (_view(out[m + "_" + n], m_at[i], L, H, D, "tok")[cut] for m in ("m1", "m2"))
            m1.mul_(b1).add_((1 - b1) * gr)
            m2.mul_(b2).add_((1 - b2) * gr * gr)
            x.sub_(rate * (m1 / (1 - b1 ** (s + 1))) / ((m2 / (1 - b2 ** (s + 1))).sqrt() + eps))
    return out


def exact(case, seed):
    if case["kind"] == "adam":
        return _exact_adam(case, seed)
    return _exact_decode(case, seed) if case["kind"] == "decode" else _exact_attn(case, seed)
