"""GPU parity of the paged short-query / decode attention (cas_paged_decode_fwd)
against the fp64 oracle: requests over retrieved cartridges held in a
paged KV pool (paper: Section "Inference", paragraph "Cartridge RAG"; the
appendix on cartridge sizes for the 16-token pages).

Bars as for the other bf16 paths: max |gpu - oracle| / max |oracle| <= 2e-2
on O, LSE absolute error <= 1e-3; every output element is compared.
"""
import numpy as np
import pytest

import oracle
from casgen import rng
from gpu_util import LSE_TOL, TOL, host, rel_err

pytestmark = pytest.mark.gpu


def _pool(seed, n_carts, cart_pages, P, Hkv, D, reqs, own_extra=0):
    """A page pool: cartridge c owns pages [c * cart_pages, (c+1) * cart_pages);
    each request's own tokens get fresh pages after them. reqs: (cartridge ids,
    own tokens, queries). Returns pool arrays (bf16 values as float32), the
    per-request key counts, query counts and page lists."""
    own_pages = [-(-own // P) for _, own, _ in reqs]
    npages = n_carts * cart_pages + sum(own_pages) + own_extra
    shape = (npages, P, Hkv, D)
    bits = lambda tag: rng.f64_to_bf16_bits(rng.normal(rng.stream_key(seed, tag), int(np.prod(shape)), 0.5))
    kp = rng.bf16_bits_to_f32(bits(1)).reshape(shape)
    vp = rng.bf16_bits_to_f32(bits(2)).reshape(shape)
    nxt = n_carts * cart_pages
    kv_lens, q_counts, pages = [], [], []
    for (carts, own, n), op in zip(reqs, own_pages):
        pl = [c * cart_pages + j for c in carts for j in range(cart_pages)]
        pl += list(range(nxt, nxt + op))
        nxt += op
        pages.append(pl)
        kv_lens.append(len(carts) * cart_pages * P + own)
        q_counts.append(n)
    return kp, vp, kv_lens, q_counts, pages


def _run(kp, vp, kv_lens, q_counts, pages, Hkv, g, D, seed, scale=None, workspace=None):
    import torch
    import paper_2606_04557_amd as cas
    Tq, Hq = sum(q_counts), Hkv * g
    q = rng.bf16_bits_to_f32(rng.f64_to_bf16_bits(rng.normal(rng.stream_key(seed, 3), Tq * Hq * D, 1.0))).reshape(
        Tq, Hq, D)
    scale = scale or float(np.float32(1.0 / np.sqrt(D)))
    dq = torch.from_numpy(q).to(torch.bfloat16).cuda()
    dk = torch.from_numpy(kp).to(torch.bfloat16).cuda()
    dv = torch.from_numpy(vp).to(torch.bfloat16).cuda()
    o, lse = cas.paged_decode_fwd(dq, dk, dv, q_counts, kv_lens, pages, Hkv, g, scale, workspace=workspace)
    torch.cuda.synchronize()
    O, LSE = oracle.paged_decode_forward(q, kp, vp, q_counts, kv_lens, pages, scale, g)
    e_o = rel_err(host(o), O)
    e_l = float(np.abs(host(lse) - LSE).max())
    print(f"decode O {e_o:.2e} LSE {e_l:.2e}")
    assert e_o <= TOL["bf16"] and e_l <= LSE_TOL["bf16"], (e_o, e_l)
    return o, lse


CASES = [
    # (page size, kv heads, group, head dim, cartridges of the pool, pages per cartridge,
    #  requests: (cartridge ids, own tokens, queries))
    dict(name="p16_decode", P=16, Hkv=8, g=4, D=128, n_carts=6, cart_pages=8,
         reqs=[([0, 3], 1, 1), ([5], 17, 1), ([1, 2, 4, 0], 40, 1), ([], 9, 1), ([2], 100, 3)]),
    # 9 queries x 4 heads = 36 rows: two row blocks; an own part that starts mid-page
    dict(name="p16_multirow", P=16, Hkv=2, g=4, D=128, n_carts=3, cart_pages=20,
         reqs=[([0, 1, 2], 61, 9), ([1], 8, 8), ([2, 0], 33, 2)]),
    dict(name="p32_d64", P=32, Hkv=2, g=2, D=64, n_carts=4, cart_pages=5,
         reqs=[([3, 1], 31, 1), ([0], 1, 1), ([2, 3, 0, 1], 64, 5)]),
    dict(name="p64_g8", P=64, Hkv=1, g=8, D=128, n_carts=2, cart_pages=3,
         reqs=[([1, 0], 70, 4), ([0], 2, 2)]),
    dict(name="p128", P=128, Hkv=4, g=4, D=128, n_carts=2, cart_pages=2,
         reqs=[([0, 1], 300, 1), ([1], 5, 5)]),
]


@pytest.mark.parametrize("case", CASES, ids=[c["name"] for c in CASES])
def test_decode_small(case):
    c = dict(case)
    kp, vp, kl, qc, pages = _pool(900 + len(c["name"]), c["n_carts"], c["cart_pages"], c["P"], c["Hkv"], c["D"],
                                  c["reqs"], own_extra=3)
    _run(kp, vp, kl, qc, pages, c["Hkv"], c["g"], c["D"], 950 + len(c["name"]))


@pytest.mark.parametrize("D,P,g", [(128, 16, 1), (64, 32, 1), (128, 64, 3)])
def test_decode_row_block_edges(D, P, g):
    """Row counts n * g around the edges of the 16- and 32-row blocks of one
    workgroup (and key counts around the 32-key tiles), mixed in one call with
    a one-token request; then each count alone, where the block size is chosen
    for it."""
    counts = [n for n in (1, 5, 6, 10, 11, 15, 16, 17, 21, 31, 32, 33, 49) if n * g <= 100]
    reqs = [([i % 3], max(n, 1 + 31 * (i % 4)), n) for i, n in enumerate(counts)]
    kp, vp, kl, qc, pages = _pool(1200 + D + g, 3, 4, P, 2, D, reqs, own_extra=1)
    _run(kp, vp, kl, qc, pages, 2, g, D, 1210 + g)
    for i in (0, 6, 7, len(counts) - 1):
        _run(kp, vp, kl[i:i + 1], qc[i:i + 1], pages[i:i + 1], 2, g, D, 1220 + i)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("keys", [255, 257, 700, 2030, 2100, 4097, 4400])
def test_decode_split_merge(D, keys):
    """One request alone: the key axis in 1 to 18 splits (8 tiles of 32 keys
    each), around the split counts at which the merge shares a row between
    more lane groups; a second, unsplit request in the same call."""
    reqs = [([], keys, 1), ([], 9, 1)]
    kp, vp, kl, qc, pages = _pool(1300 + keys, 0, 0, 16, 2, D, reqs)
    _run(kp, vp, kl, qc, pages, 2, 4, D, 1301)


def _shared_problem(seed, P, D, Hkv, g, n_req, n_carts, cart_keys, pick, new, own, cut=None):
    """Requests that share cartridges of cart_keys keys: request r reads the
    cartridges pick(r) and own(r) tokens of its own, of which new(r) are
    queries. cut(r): pages dropped from the end of its last cartridge."""
    cp = cart_keys // P
    reqs, pages, kv = [], [], []
    nxt = n_carts * cp
    for r in range(n_req):
        ids = [c * cp + j for c in pick(r) for j in range(cp)]
        if cut:
            ids = ids[: len(ids) - cut(r)]
        op = -(-own(r) // P)
        pages.append(ids + list(range(nxt, nxt + op)))
        nxt += op
        kv.append(len(ids) * P + own(r))
    shape = (nxt, P, Hkv, D)
    bits = lambda tag: rng.f64_to_bf16_bits(rng.normal(rng.stream_key(seed, tag), int(np.prod(shape)), 0.5))
    kp = rng.bf16_bits_to_f32(bits(1)).reshape(shape)
    vp = rng.bf16_bits_to_f32(bits(2)).reshape(shape)
    return kp, vp, kv, [new(r) for r in range(n_req)], pages


SHARED = [
    # every request reads the same cartridge first, then one of two others; ends off the page
    dict(name="prefix", P=16, D=128, Hkv=2, g=4, n_req=9, n_carts=3, cart_keys=512, pick=lambda r: [0, 1 + r % 2],
         new=lambda r: 1, own=lambda r: 1 + 7 * r),
    # more than 32 rows of readers per run; a request that reads a cartridge twice, one that reads none
    dict(name="many_twice", P=32, D=64, Hkv=1, g=5, n_req=12, n_carts=4, cart_keys=320,
         pick=lambda r: [] if r == 3 else [2, 2] if r == 5 else [r % 4, (r + 1) % 4, 2][: 1 + r % 3],
         new=lambda r: 1 + r % 3, own=lambda r: 3 + r),
    # runs cut short by one reader; no own tokens past the queries, so a run's last pages hold a reader's queries
    dict(name="cut", P=16, D=128, Hkv=8, g=4, n_req=6, n_carts=2, cart_keys=1024, pick=lambda r: [r % 2, 1 - r % 2],
         new=lambda r: 1, own=lambda r: 0 if r % 2 else 40, cut=lambda r: r),
    # large pages, runs split into pieces, the last tile of a piece partly past the run
    dict(name="pieces", P=128, D=128, Hkv=1, g=2, n_req=5, n_carts=2, cart_keys=2048, pick=lambda r: [0, 1],
         new=lambda r: 2, own=lambda r: 2 + 100 * r),
    # few readers: their rows fit one 16-row block
    dict(name="few", P=16, D=128, Hkv=2, g=4, n_req=3, n_carts=2, cart_keys=768, pick=lambda r: [0, 1] if r else [0],
         new=lambda r: 1, own=lambda r: 3 + 9 * r),
    # below the shortest run worth sharing (in an order in which no two cartridges' page ids continue each other)
    dict(name="short", P=16, D=64, Hkv=2, g=2, n_req=8, n_carts=3, cart_keys=128, pick=lambda r: [0, 2, 1],
         new=lambda r: 1, own=lambda r: 5),
]


@pytest.mark.parametrize("case", SHARED, ids=[c["name"] for c in SHARED])
def test_decode_shared_runs(case):
    """Cartridges that several requests read are streamed once for all of
    them: each request's output still equals its own gathered keys."""
    c = dict(case)
    c.pop("name")
    Hkv, g, D = c["Hkv"], c["g"], c["D"]
    kp, vp, kl, qc, pages = _shared_problem(1400, **c)
    _run(kp, vp, kl, qc, pages, Hkv, g, D, 1401)


def test_decode_shared_runs_in_a_workspace_without_room_for_them():
    """A workspace that holds only the plan that shares nothing is used for that plan."""
    import ctypes
    import torch
    import paper_2606_04557_amd as cas
    c = dict(SHARED[1])
    c.pop("name")
    Hkv, g, D, P = c["Hkv"], c["g"], c["D"], c["P"]
    kp, vp, kl, qc, pages = _shared_problem(1450, **c)
    ends = np.cumsum([0] + [len(pl) for pl in pages])
    private = cas.DecodeProblem(qc, kl, [list(range(a, b)) for a, b in zip(ends, ends[1:])], int(ends[-1]), P, Hkv, g, D, 0.1)
    n = ctypes.c_size_t(0)
    cas._check(cas.load().cas_paged_decode_workspace_size(ctypes.byref(private.c), ctypes.byref(n)))
    assert n.value < cas.decode_plan(cas.DecodeProblem(qc, kl, pages, kp.shape[0], P, Hkv, g, D, 0.1))[0].ws_bytes
    ws = torch.full((n.value + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    _run(kp, vp, kl, qc, pages, Hkv, g, D, 1451, workspace=ws[:n.value])
    assert bool((ws[n.value:] == 0x5a).all())


@pytest.mark.parametrize("n_req", [1, 2, 6])
def test_decode_nan_key_stays(n_req):
    """A key that is not a number makes every row that reads it NaN, whether the
    row's keys take one pass (two requests of 148 keys), several pieces (one of
    2,612) or a run shared with other requests, in O and in LSE, and leaves the other
    requests alone."""
    import torch
    import paper_2606_04557_amd as cas
    own = 2100 if n_req == 1 else 20
    reqs = [([0, 1] if n_req > 2 and r % 2 else [0], own, 1) for r in range(n_req)] + [([], 700, 1)]
    kp, vp, kl, qc, pages = _pool(1500 + n_req, 2, 8 if n_req == 2 else 32, 16, 2, 128, reqs)
    plan = cas.decode_plan(cas.DecodeProblem(qc, kl, pages, kp.shape[0], 16, 2, 4, 128, 0.1))
    assert (plan[0].shared_runs > 0) == (n_req == 6) and any(r[2] < 0 for r in plan[1]) == (n_req == 2)
    o, lse = _run(kp, vp, kl, qc, pages, 2, 4, 128, 1501)
    good, good_lse = o.clone(), lse.clone()
    kp = kp.copy()
    kp[5, 3, 1, 7] = np.nan          # cartridge 0, KV head 1
    q = rng.bf16_bits_to_f32(rng.f64_to_bf16_bits(rng.normal(rng.stream_key(1501, 3), sum(qc) * 8 * 128, 1.0)))
    q = torch.from_numpy(q.reshape(sum(qc), 8, 128)).to(torch.bfloat16).cuda()
    o, lse = cas.paged_decode_fwd(q, torch.from_numpy(kp).to(torch.bfloat16).cuda(), torch.from_numpy(vp).to(torch.bfloat16).cuda(),
                                qc, kl, pages, 2, 4, float(np.float32(1.0 / np.sqrt(128))))
    torch.cuda.synchronize()
    assert bool(torch.isnan(o[:-1, 4:]).all())
    assert torch.equal(o[:-1, :4], good[:-1, :4]) and torch.equal(o[-1], good[-1])
    assert bool(torch.isnan(lse[4:, :-1]).all())
    assert torch.equal(lse[:4, :-1], good_lse[:4, :-1]) and torch.equal(lse[:, -1], good_lse[:, -1])


def test_decode_retrieval_mix_full_size():
    """Cartridge-RAG decode step at full size: a pool of 256 cartridges of 1,024
    tokens (16,384 pages of 16 tokens, 8 KV heads x 128); 64 requests, each over
    4 retrieved cartridges plus its own 64-token prompt, decoding one token
    (kv_len = 4,161). Every output is compared."""
    sel = [rng.choose_distinct(rng.stream_key(5, 8, r), 256, 4) for r in range(64)]
    reqs = [(s, 65, 1) for s in sel]
    kp, vp, kl, qc, pages = _pool(77, 256, 64, 16, 8, 128, reqs)
    _run(kp, vp, kl, qc, pages, 8, 4, 128, 78)


def test_decode_rejects_bad_tables():
    import torch
    import paper_2606_04557_amd as cas
    kp = torch.zeros((4, 16, 2, 64), dtype=torch.bfloat16, device="cuda")
    q = torch.zeros((2, 4, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(cas.CasError):       # page id out of range
        cas.paged_decode_fwd(q, kp, kp.clone(), [1, 1], [20, 3], [[0, 4], [1]], 2, 2, 0.125)
    with pytest.raises(cas.CasError):       # page count != ceil(kv_len / page_size)
        cas.paged_decode_fwd(q, kp, kp.clone(), [1, 1], [20, 3], [[0], [1]], 2, 2, 0.125)
    with pytest.raises(cas.CasError):       # more queries than keys
        cas.paged_decode_fwd(q, kp, kp.clone(), [2, 0], [1, 3], [[0], [1]], 2, 2, 0.125)


def test_decode_pool_beyond_4gib():
    """Pages past the first 4 GiB of a 5 GB pool (page ids above 16,384 with
    256 KiB pages: 128 tokens x 8 KV heads x 128): every page address is
    computed in 64 bits. Only the listed pages hold data; the oracle reads a
    compact copy of them under renumbered ids. Every output is compared."""
    import torch
    import paper_2606_04557_amd as cas
    P, Hkv, g, D = 128, 8, 4, 128
    n_pool = 20_000                               # 20,000 x 256 KiB = 5.2 GB per tensor
    reqs = [(3, 300, 1), (2, 129, 3), (4, 1, 1)]   # (pages, tokens in the last page, queries)
    ids, kv_lens, q_counts = [], [], []
    nxt = 16_380
    for npg, last, nq in reqs:
        ids.append(list(range(nxt, nxt + npg)))
        nxt += npg + 997                          # scattered, and all but the first few past 2^32 bytes
        kv_lens.append((npg - 1) * P + min(last, P))
        q_counts.append(nq)
    used = sorted({i for r in ids for i in r})
    assert max(used) < n_pool and max(used) * P * Hkv * D * 2 > 2 ** 32
    shape = (len(used), P, Hkv, D)
    bits = lambda tag: rng.f64_to_bf16_bits(rng.normal(rng.stream_key(991, tag), int(np.prod(shape)), 0.5))
    kc = rng.bf16_bits_to_f32(bits(1)).reshape(shape)
    vc = rng.bf16_bits_to_f32(bits(2)).reshape(shape)
    kp = torch.empty((n_pool, P, Hkv, D), dtype=torch.bfloat16, device="cuda")
    vp = torch.empty_like(kp)
    idx = torch.tensor(used, device="cuda")
    kp[idx] = torch.from_numpy(kc).to(torch.bfloat16).cuda()
    vp[idx] = torch.from_numpy(vc).to(torch.bfloat16).cuda()
    Tq, Hq = sum(q_counts), Hkv * g
    q = rng.bf16_bits_to_f32(rng.f64_to_bf16_bits(rng.normal(rng.stream_key(992, 3), Tq * Hq * D, 1.0))).reshape(
        Tq, Hq, D)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    o, lse = cas.paged_decode_fwd(torch.from_numpy(q).to(torch.bfloat16).cuda(), kp, vp, q_counts, kv_lens, ids,
                                  Hkv, g, scale)
    torch.cuda.synchronize()
    remap = {p: i for i, p in enumerate(used)}
    O, LSE = oracle.paged_decode_forward(q, kc, vc, q_counts, kv_lens, [[remap[i] for i in r] for r in ids], scale, g)
    e_o = rel_err(host(o), O)
    e_l = float(np.abs(host(lse) - LSE).max())
    print(f"pool past 4 GiB: O {e_o:.2e} LSE {e_l:.2e}")
    assert e_o <= TOL["bf16"] and e_l <= LSE_TOL["bf16"], (e_o, e_l)
    del kp, vp
    torch.cuda.empty_cache()
