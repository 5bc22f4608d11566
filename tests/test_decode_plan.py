"""The launch plan of the paged decode (pure host): every query row sees each of
its keys exactly once, every partial has its own place, and page runs that
requests share are streamed once where that saves work."""
import os
import random

import pytest

from test_gpu_decode import SHARED, _shared_problem

TILE = 32


@pytest.fixture(scope="module")
def cas():
    import paper_2606_04557_amd as cas
    cas.load()
    return cas


def problem(cas, q, kv, pages, P=16, Hkv=2, g=2, D=64):
    npages = max((x for pl in pages for x in pl), default=0) + 1
    return cas.DecodeProblem(q, kv, pages, npages, P, Hkv, g, D, 0.125)


def check(cas, q, kv, pages, P=16, Hkv=2, g=2, D=64):
    """Walks the plan's workgroups and compares what each (token, head) sees
    with its request's own key list."""
    info, rows, work = cas.decode_plan(problem(cas, q, kv, pages, P, Hkv, g, D))
    ids = [x for pl in pages for x in pl]
    Hq = Hkv * g
    seen, parts = {}, {}
    assert sum(w[5] - w[4] for w in work) == info.key_tiles
    assert [w[5] - w[4] for w in work] == sorted((w[5] - w[4] for w in work), reverse=True)
    for page0, nkeys, full, kvh, t0, t1, row0, nrows, piece in work:
        assert 0 <= t0 < t1 <= -(-nkeys // TILE) and 1 <= nrows <= 16 * info.row_blocks and 0 <= kvh < Hkv
        assert 0 <= row0 and row0 + nrows <= info.num_rows and page0 + -(-nkeys // P) <= len(ids)
        for base, lim, part in rows[row0: row0 + nrows]:
            assert full <= lim < nkeys
            k = (base, kvh)
            seen.setdefault(k, []).extend(ids[page0 + i // P] * P + i % P for i in range(t0 * TILE, min(t1 * TILE, lim + 1)))
            parts.setdefault(k, []).append(part + piece if part >= 0 else -1)
    tok = 0
    for n, L, pl in zip(q, kv, pages):
        keys = [pl[i // P] * P + i % P for i in range(L)]
        for i in range(n):
            want = sorted(keys[: L - n + i + 1])
            for h in range(g):
                for kvh in range(Hkv):
                    k = ((tok + i) * Hq + h, kvh)
                    assert sorted(seen.pop(k)) == want
                    p = sorted(parts[k])
                    assert p == ([-1] if len(p) == 1 else list(range(len(p)))) and len(p) <= info.max_partials
        tok += n
    assert not seen and info.max_partials <= 64
    return info


def draw(r):
    """Requests over a pool of consecutive pages: cartridges, parts of them,
    repeated, reordered and cut ones, scattered pages, own pages of any count."""
    P = r.choice([16, 16, 32, 64, 128])
    n_carts, cp = r.randint(1, 6), r.randint(1, 6 * 256 // P // 2)
    q, kv, pages = [], [], []
    nxt = n_carts * cp
    forks = []
    for _ in range(r.randint(1, 9)):
        pl = []
        for _ in range(r.randint(0, 5)):
            c = r.randrange(n_carts)
            a, b = (0, cp) if r.random() < 0.6 else sorted((r.randint(0, cp), r.randint(0, cp)))
            run = list(range(c * cp + a, c * cp + b))
            if r.random() < 0.1:
                r.shuffle(run)
            pl += run
        if forks and r.random() < 0.3:
            pl = list(r.choice(forks))
        n = r.choice([1, 1, 2, 5, 9])
        own = r.choice([0, 1, 7, P, 3 * P + 1])
        op = -(-own // P)
        pl += range(nxt, nxt + op)
        nxt += op
        L = len(pl) * P - (op * P - own)
        if L < n:
            pl, L = pl + [nxt], len(pl) * P + n
            nxt += 1
        forks.append(pl[: L // P])
        q.append(n)
        kv.append(L)
        pages.append(pl)
    return q, kv, pages, P, r.randint(1, 3), r.choice([1, 3, 4, 8]), r.choice([64, 128])


@pytest.mark.parametrize("seed", range(300))
def test_each_key_once(cas, seed):
    check(cas, *draw(random.Random(seed)))


RUNS = dict(prefix=3, many_twice=4, cut=2, pieces=1, few=2, short=0)


@pytest.mark.parametrize("case", SHARED, ids=[c["name"] for c in SHARED])
def test_shared_cases_share(cas, case):
    """The plans that the GPU tests of shared runs take do share (and the one
    with runs below the limit does not)."""
    c = dict(case)
    name = c.pop("name")
    Hkv, g, D, P = c["Hkv"], c["g"], c["D"], c["P"]
    _, _, kv, q, pages = _shared_problem(1400, **c)
    info = check(cas, q, kv, pages, P, Hkv, g, D)
    assert info.shared_runs == RUNS[name]
    assert info.row_blocks == (1 if name in ("few", "short") else 2)


@pytest.mark.parametrize("Hkv", [1, 2, 4, 8])
@pytest.mark.parametrize("keys", [1024, 16384, 32768, 60000, 65536, 250000])
@pytest.mark.parametrize("n_req", [2, 8, 16])
def test_one_run_of_any_length_is_streamed_once(cas, Hkv, keys, n_req):
    """One-token requests over one run of pages and a few keys of their own:
    the run is streamed once per 32 rows of its readers however long it is,
    and no request has more than 64 partials."""
    P, g, own = 16, 4, 50
    run = list(range(keys // P))
    op = -(-own // P)
    pages = [run + [len(run) + r * op + j for j in range(op)] for r in range(n_req)]
    kv = [len(run) * P + own] * n_req
    info, _, _ = cas.decode_plan(problem(cas, [1] * n_req, kv, pages, P, Hkv, g, 128))
    assert info.shared_runs == 1 and info.max_partials <= 64
    # Once per 32 rows, the own keys per request; a piece's last tile may be partly past the run.
    assert info.key_tiles == Hkv * (-(-n_req * g // 32) * -(-len(run) * P // TILE) + n_req * -(-own // TILE))
    if keys <= 16384:
        check(cas, [1] * n_req, kv, pages, P, Hkv, g, 128)


@pytest.mark.parametrize("many", [60, 63, 64, 65, 70, 100])
def test_a_request_over_too_many_runs_reads_alone(cas, many):
    """15 requests over the same 4 cartridges and two over `many` others: past
    64 partials each (the runs and its own keys) these two read their keys by
    themselves, and the others still share."""
    P, cp, Hkv = 16, 16, 2
    cart = lambda c: [c * cp + j for j in range(cp)]
    pages = [sum((cart(2 * c + 1) for c in range(4)), []) for _ in range(15)]
    pages += [sum((cart(2 * c) for c in range(many)), []) for _ in range(2)]
    kv = [len(pl) * P + 13 for pl in pages]
    for r, pl in enumerate(pages):
        pl.append(2 * cp * many + r)
    info = check(cas, [1] * 17, kv, pages, P, Hkv, 4, 64)
    shared = 4 * 8 * -(-60 // (16 * info.row_blocks)) + 15   # 60 rows; a tile of their own each
    wide = many * 8 + 2 if many < 64 else 2 * (many * 8 + 1)
    assert info.key_tiles == Hkv * (shared + wide)
    assert info.shared_runs == (4 + many if many < 64 else 4)


def test_a_request_over_the_whole_pool_reads_alone(cas):
    """Eight requests in pairs over 20 cartridges each, and one whose pages are
    the whole pool in one stretch: it holds 80 runs and reads alone, the pairs share."""
    P, cp, Hkv = 16, 16, 2
    pages = [[(40 * (r // 2) + 2 * c) * cp + j for c in range(20) for j in range(cp)] for r in range(8)]
    pages.append(list(range(160 * cp)))
    kv = [len(pl) * P + 13 for pl in pages]
    for r, pl in enumerate(pages):
        pl.append(160 * cp + r)
    info = check(cas, [1] * 9, kv, pages, P, Hkv, 4, 64)
    assert info.shared_runs == 80
    assert info.key_tiles == Hkv * (80 * 8 + 8 + 160 * 8 + 1)


def plan_us(cas, pages, own=65, P=16):
    import ctypes
    import time
    nxt = max(x for pl in pages for x in pl) + 1
    kv = [len(pl) * P + own for pl in pages]
    op = -(-own // P)
    pages = [pl + list(range(nxt + b * op, nxt + (b + 1) * op)) for b, pl in enumerate(pages)]
    prob = cas.DecodeProblem([1] * len(pages), kv, pages, nxt + len(pages) * op, P, 8, 4, 128, 0.1)
    n, best = ctypes.c_size_t(0), 1e9
    for _ in range(150):
        t = time.perf_counter()
        assert cas.load().cas_paged_decode_workspace_size(ctypes.byref(prob.c), ctypes.byref(n)) == 0
        best = min(best, time.perf_counter() - t)
    return best * 1e6


@pytest.mark.parametrize("name,bound", [("scattered", 2.0), ("20 of 80", 8.0), ("60 of 80", 9.0), ("70 of 80", 5.0)])
def test_plan_time(cas, name, bound):
    """Looking for shared runs costs little beside reading the page lists: the
    best plan time of 64 requests against that of as many private pages in one
    stretch each. Measured 0.8, 4.0, 5.5 and 2.7 times (a search that sorted
    every stretch's ends and compared 16 ids at every page: 3.3, 13, 19 and 10)."""
    if os.environ.get("CAS_LIB"):
        pytest.skip("times the library as it is built for use")
    r = random.Random(3)
    if name == "scattered":
        k = 256
        ids = list(range(64 * k))
        r.shuffle(ids)
        pages = [ids[b * k:(b + 1) * k] for b in range(64)]
    else:
        k = 16 * int(name.split()[0])
        pages = [[c * 16 + j for c in r.sample(range(80), k // 16) for j in range(16)] for _ in range(64)]
    private = [list(range(b * (k + 1), b * (k + 1) + k)) for b in range(64)]
    ratio = plan_us(cas, pages) / plan_us(cas, private)
    print(f"{name}: {ratio:.2f}")
    assert ratio <= bound


@pytest.mark.parametrize("n,given", [(4, None), (12, None), (60, None), (60, 1 << 16), (4, 0)])
def test_a_problem_is_planned_once(cas, monkeypatch, n, given):
    """Without a workspace, or with one that is too small, a decode call plans
    its problem once, whatever it shares, and offers what it needs and no more;
    further calls on the same DecodeProblem plan nothing."""
    import torch
    from paper_2606_04557_amd import _lib
    real, plans, offered = cas.load(), [], []

    class Lib:
        def __getattr__(self, name):
            assert name in ("cas_paged_decode_plan_destroy", "cas_paged_decode_plan_matches", "cas_last_error_message",
                            "cas_status_string"), name
            return getattr(real, name)

        def cas_paged_decode_plan_create(self, prob, handle, nbytes):
            status = real.cas_paged_decode_plan_create(prob, handle, nbytes)
            plans.append(nbytes._obj.value)
            return status

        def cas_paged_decode_run(self, handle, q, k, v, o, lse, ws, nbytes, stream):
            offered.append(nbytes)
            return _lib.CAS_OK

    monkeypatch.setattr(cas, "load", lambda: Lib())
    monkeypatch.setattr(cas, "_stream_handle", lambda device, stream: None)
    r = random.Random(9)
    pages = [[c * 16 + j for c in r.sample(range(80), n) for j in range(16)] + [1280 + b] for b in range(64)]
    q = torch.zeros(64, 4, 64, dtype=torch.bfloat16)
    pool = torch.zeros(1344, 16, 2, 64, dtype=torch.bfloat16)
    kv = [len(pl) * 16 - 3 for pl in pages]
    ws = torch.empty(given, dtype=torch.uint8) if given is not None else None
    call = lambda prob: cas.paged_decode_fwd(q, pool, pool.clone(), [1] * 64, kv, pages, 2, 2, 0.125, problem=prob, workspace=ws)
    prob = problem(cas, [1] * 64, kv, pages)
    for _ in range(3):
        call(prob)
        assert len(plans) == 1 and offered[-1] == plans[0]
    call(None)
    assert len(plans) == 2 and offered[-1] == plans[1]


def fwd_status(cas, prob, nbytes):
    """What a call with a workspace of nbytes at an odd address says, planned
    before or not: too small, or (large enough, and refused for the address
    before any device is touched) misaligned."""
    import ctypes
    A = 1 << 44
    args = A, 2 * A, 3 * A, 4 * A, None, 5 * A + 4, nbytes, None
    status = cas.load().cas_paged_decode_fwd(ctypes.byref(prob.c), *args)
    assert cas.load().cas_paged_decode_run(prob.plan().handle, *args) == status
    return status


@pytest.mark.parametrize("seed", range(40))
def test_workspace_serves_other_pages_of_the_same_lengths(cas, seed):
    """A workspace of the size asked for with one set of page ids is accepted
    with any other of the same counts and lengths, shared or not, and a byte
    less than the smaller of the two plans is not."""
    import ctypes
    from paper_2606_04557_amd import _lib
    r = random.Random(700 + seed)
    q, kv, pages, P, Hkv, g, D = draw(r)
    n = sum(len(pl) for pl in pages)
    ids, private = list(range(n)), []
    for pl in pages:
        private.append(ids[: len(pl)])
        del ids[: len(pl)]
    r.shuffle(pages[0])
    same = [list(range(len(pl))) for pl in pages]
    sizes, probs = [], []
    for pls in (pages, private, same):
        probs.append(problem(cas, q, kv, pls, P, Hkv, g, D))
        out = ctypes.c_size_t(0)
        assert cas.load().cas_paged_decode_workspace_size(ctypes.byref(probs[-1].c), ctypes.byref(out)) == _lib.CAS_OK
        sizes.append(out.value)
    assert sizes[1] <= min(sizes)
    for prob in probs:
        for s in sizes:
            assert fwd_status(cas, prob, s) == _lib.CAS_ERR_ALIGNMENT
        plan = cas.decode_plan(prob)[0].ws_bytes
        assert fwd_status(cas, prob, min(plan, sizes[1]) - 1) == _lib.CAS_ERR_WORKSPACE
        assert cas.load().cas_last_workspace_needed() == sizes[probs.index(prob)]


def test_plan_handle_validation(cas):
    import ctypes
    from paper_2606_04557_amd import _lib
    lib, h, n = cas.load(), ctypes.c_void_p(), ctypes.c_size_t(0)
    bad = problem(cas, [1], [17], [[0]])     # 17 keys need two pages of 16
    assert lib.cas_paged_decode_plan_create(ctypes.byref(bad.c), ctypes.byref(h), ctypes.byref(n)) == _lib.CAS_ERR_INVALID_ARGUMENT
    assert not h.value and lib.cas_paged_decode_plan_destroy(None) == _lib.CAS_OK
    with pytest.raises(cas.CasError):
        bad.plan()
    A = 1 << 44
    assert lib.cas_paged_decode_run(None, A, A, A, A, None, A, 1 << 20, None) == _lib.CAS_ERR_INVALID_ARGUMENT
    good = problem(cas, [1], [17], [[0, 1]])
    run = lambda *a: lib.cas_paged_decode_run(good.plan().handle, *a)
    assert run(None, A, 2 * A, 3 * A, None, 4 * A, 1 << 20, None) == _lib.CAS_ERR_INVALID_ARGUMENT
    assert run(A, 2 * A, 3 * A, A, None, 4 * A, 1 << 20, None) == _lib.CAS_ERR_INVALID_ARGUMENT      # o over q
    assert run(A + 8, 2 * A, 3 * A, 4 * A, None, 5 * A, 1 << 20, None) == _lib.CAS_ERR_ALIGNMENT
    assert run(A, 2 * A, 3 * A, 4 * A, None, None, 0, None) == _lib.CAS_ERR_WORKSPACE
    assert lib.cas_last_workspace_needed() == good.plan().ws_bytes


def test_plan_keeps_its_own_tables(cas):
    """A plan does not look at the caller's tables again: freed or changed, they
    neither take a run out of the pool nor change what it needs."""
    import ctypes
    from paper_2606_04557_amd import _lib
    r = random.Random(5)
    pages = [[c * 16 + j for c in r.sample(range(80), 20) for j in range(16)] for _ in range(64)]
    prob = problem(cas, [1] * 64, [len(pl) * 16 - 3 for pl in pages], pages)
    lib, h, n = cas.load(), ctypes.c_void_p(), ctypes.c_size_t(0)
    info = cas.decode_plan(prob)[0]
    assert info.shared_runs > 0 and lib.cas_paged_decode_plan_create(ctypes.byref(prob.c), ctypes.byref(h), ctypes.byref(n)) == 0
    for a in (prob._qo, prob._kv, prob._po, prob._ids):
        for i in range(len(a)):
            a[i] = -7
    A = 1 << 44
    run = lambda nbytes: lib.cas_paged_decode_run(h, A, 2 * A, 3 * A, 4 * A, None, 5 * A + 4, nbytes, None)
    # (Large enough and refused for its address; the smaller one is for the plan that shares nothing, made by the run.)
    assert run(n.value) == run(info.ws_bytes - 1) == _lib.CAS_ERR_ALIGNMENT
    assert lib.cas_paged_decode_plan_destroy(h) == _lib.CAS_OK


def test_a_changed_problem_is_planned_again(cas):
    """A DecodeProblem whose tables or values change after its first call is
    planned anew (and validated: a page id past the pool is refused)."""
    prob = problem(cas, [1, 1], [40, 33], [[0, 1, 2], [3, 4, 5]])
    for table, i, to in (("_kv", 0, 41), ("_ids", 5, 2), ("_po", 0, 0), ("_qo", 1, 1)):
        plan = prob.plan()
        assert prob.plan() is plan
        a = getattr(prob, table)
        changed, a[i] = a[i] != to, to
        assert (prob.plan() is not plan) == changed
    for name, to in (("softmax_scale", 0.25), ("num_pages", 7), ("batch", 1), ("group_size", 1), ("num_kv_heads", 1),
                     ("head_dim", 128)):
        plan = prob.plan()
        setattr(prob.c, name, to)
        assert prob.plan() is not plan and prob.plan() is prob.plan()
    prob._ids[0] = 7
    with pytest.raises(cas.CasError):
        prob.plan()
