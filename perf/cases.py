"""What a serving program asks of this library, as cases that can be timed and compared.

A case is a dict of plain values; its "kind" names the call sequence of one pass:

  step    emb_lookup of the new tokens' features, then hstu_step over a batch of requests (prefill, or new tokens behind a
          cached history)
  loop    the same for one turn of a serving loop: the KV bookkeeping calls of every request, the page tables that follow
          from them, lookups, step; returning users append to their cached history, new ones recompute theirs
  lookup  emb_lookup / emb_lookup_noalloc alone, with everything resident or with a cache smaller than the working set
  tables  emb_lookup_tables over several tables of different widths
  split   one excursion of the EMB:KV boundary: shrink, lookups, growth, refill of the new ways

Only public entry points are called.  Inputs come from the seed: Zipf-like ids, lognormal history lengths and time gaps,
random weights, random cached keys and values.
"""
import math
import statistics

import numpy as np
import torch

from paper_2605_04450_amd import binding as B
from paper_2605_04450_amd import device as D
from paper_2605_04450_amd import synth

N_TIME = 32
TIMELINES = 64
REFILL_CHUNK = 1 << 18


# ---- cases ------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the small fp32 configuration: prefill of four short requests
        dict(name="step_fp32_small", kind="step", dtype="fp32", L=1, d=64, H=2, page_tokens=16, requests=4, cached=0,
             new=256, spread=0.0, bag=1, rows=100_000, zipf=1.0),
        # one user comes back: 64 new tokens behind one cached history, the latency of a single request
        dict(name="step_append_one", kind="step", dtype="bf16", L=4, d=256, H=4, page_tokens=64, requests=1, cached=2973,
             new=64, spread=0.0, bag=8, rows=200_000, zipf=0.9),
        # a batch of returning users
        dict(name="step_append_batch", kind="step", dtype="bf16", L=4, d=256, H=4, page_tokens=64, requests=128, cached=3072,
             new=64, spread=0.6, bag=8, rows=1_000_000, zipf=0.9),
        # short ragged prefills of the narrow model, small pages, pooled features
        dict(name="step_prefill_ragged", kind="step", dtype="bf16", L=4, d=128, H=2, page_tokens=16, requests=13, cached=0,
             new=190, spread=0.9, bag=4, rows=300_000, zipf=0.9),
        # the flagship batch: 64 histories of 2048 tokens on average, computed from the start
        dict(name="step_prefill_batch", kind="step", dtype="bf16", L=4, d=256, H=4, page_tokens=64, requests=64, cached=0,
             new=2048, spread=0.6, bag=1, rows=1_000_000, zipf=1.0),
        # long cached histories of the wide model, 512 new tokens each
        dict(name="step_long_reuse", kind="step", dtype="bf16", L=8, d=512, H=8, page_tokens=64, requests=32, cached=16384,
             new=512, spread=0.0, bag=1, rows=100_000, zipf=1.0),
        # a turn of the serving loop with about 2000 users resident, half of the batch returning
        dict(name="loop_serving", kind="loop", dtype="bf16", L=4, d=256, H=4, page_tokens=64, requests=128, returning=64,
             mean=2048, new=64, kv_pages=65536, bag=8, rows=2_000_000, zipf=0.9),
        # the features of a single request
        dict(name="lookup_small", kind="lookup", call="lookup", dtype="bf16", d=256, lookups=1000, bag=1, rows=100_000,
             room=2.0, zipf=1.0, flags=False),
        # eight sum-pooled features for 256 x 1024 tokens, rows resident
        dict(name="lookup_pooled_large", kind="lookup", call="lookup", dtype="bf16", d=128, lookups=2_097_152, bag=8,
             rows=8_000_000, room=1.6, zipf=0.8, flags=False),
        # a cache that holds an eighth of the table: misses cross the host link in every batch
        dict(name="lookup_misses", kind="lookup", call="lookup", dtype="bf16", d=256, lookups=262_144, bag=1,
             rows=4_000_000, room=0.125, zipf=0.9, flags=True),
        # 24 tables of three widths probed in one launch
        dict(name="lookup_tables", kind="tables", dtype="bf16", d=128, tables=24, tokens=65_536, bag=1, rows=200_000,
             zipf=0.8),
        # the boundary moves by the controller's largest step and back, with lookups in between
        dict(name="split_and_refill", kind="split", dtype="bf16", d=256, pages=16384, low=0.44, high=0.50, lookups=65_536,
             rows=4_000_000, zipf=0.9),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw_step(rng):
    if rng.random() < 0.2:
        return dict(kind="step", dtype="fp32", L=rng.randint(1, 2), d=64, H=2, page_tokens=16, requests=log_int(rng, 1, 16),
                    cached=rng.choice([0, log_int(rng, 16, 512)]), new=log_int(rng, 8, 256), spread=rng.choice([0.0, 0.6]),
                    bag=rng.choice([1, 4]), rows=100_000, zipf=1.0)
    d = rng.choice([64, 128, 128, 256, 256, 256, 512])
    prefill = rng.random() < 0.5
    return dict(kind="step", dtype="bf16", L=rng.randint(1, 8 if d == 512 else 4), d=d, H=d // 64,
                page_tokens=rng.choice([16, 64, 64]), requests=log_int(rng, 1, 128),
                cached=0 if prefill else log_int(rng, 64, 16384), new=log_int(rng, 32, 4096) if prefill else log_int(rng, 1, 512),
                spread=rng.choice([0.0, 0.6, 0.9]), bag=rng.choice([1, 1, 4, 8]), rows=log_int(rng, 50_000, 1_000_000),
                zipf=rng.choice([0.8, 0.9, 1.0]))


def draw_loop(rng):
    requests, mean, d = log_int(rng, 8, 128), log_int(rng, 600, 2048), rng.choice([128, 256])
    return dict(kind="loop", dtype="bf16", L=4, d=d, H=d // 64, page_tokens=64, requests=requests,
                returning=rng.randint(1, requests - 1), mean=mean, new=log_int(rng, 16, 128),
                kv_pages=log_int(rng, max(8192, requests * mean // 8), 65536), bag=rng.choice([1, 4, 8]), rows=log_int(rng, 200_000, 2_000_000),
                zipf=rng.choice([0.8, 0.9, 1.0]))


def draw_lookup(rng):
    bag = rng.choice([1, 1, 2, 3, 4, 8, 16])
    d = rng.choice([32, 64, 128, 256, 256, 512])
    dtype = "fp32" if d <= 256 and rng.random() < 0.25 else "bf16"
    lookups = log_int(rng, 64, 2_097_152 if d <= 128 else 524_288)
    resident = rng.random() < 0.5
    small = lookups <= B.NOALLOC_MAX_LOOKUPS and lookups * d * (4 if dtype == "fp32" else 2) <= B.NOALLOC_MAX_ROW_BYTES_TOTAL
    rows = log_int(rng, 20_000, 4_000_000) if resident else min(4_000_000, max(20_000, lookups * rng.randint(8, 16)))
    return dict(kind="lookup", call="noalloc" if small and rng.random() < 0.3 else "lookup", dtype=dtype, d=d,
                lookups=max(1, lookups // bag) * bag, bag=bag, rows=rows, room=2.0 if resident else rng.choice([0.1, 0.2]),
                zipf=rng.choice([0.8, 0.9, 1.0]), flags=rng.random() < 0.5)


def draw_tables(rng):
    tables = rng.choice([2, 4, 8, 10, 16, 24, 25])
    return dict(kind="tables", dtype="bf16", d=rng.choice([128, 256]), tables=tables, tokens=log_int(rng, 100, 65_536),
                bag=tables if tables <= 8 and rng.random() < 0.3 else 1, rows=log_int(rng, 10_000, 100_000), zipf=0.8)


def draw_split(rng):
    high, step = rng.uniform(0.3, 0.8), rng.choice([0.02, 0.04, 0.06])
    pages = 32 * log_int(rng, 32, 512)
    slots = high * pages * 512
    return dict(kind="split", dtype="bf16", d=256, pages=pages, low=high - step, high=high, lookups=log_int(rng, 1000, 65_536),
                rows=int(min(4_000_000, slots * rng.uniform(0.8, 1.0))), zipf=0.9)


def draw(rng):
    most = [work(c) for c in listed()]
    bytes_most, flops_most = max(w["bytes"] for w in most), max(w["flops"] for w in most)
    while True:
        case = rng.choice([draw_step, draw_step, draw_step, draw_loop, draw_lookup, draw_lookup, draw_tables, draw_split])(rng)
        w = work(case)
        if w["bytes"] <= bytes_most and w["flops"] <= flops_most:
            return case


# ---- sizes ------------------------------------------------------------------------------------------------------------
def esize(case):
    return 4 if case["dtype"] == "fp32" else 2


def lengths(n, mean, spread, lo=1, hi=1 << 30):
    """n lengths with the given mean: the quantiles of a lognormal distribution (all equal without a spread)."""
    mu = math.log(mean) - 0.5 * spread * spread
    q = statistics.NormalDist().inv_cdf
    return [min(hi, max(lo, round(math.exp(mu + spread * q((i + 0.5) / n))))) for i in range(n)]


def step_lengths(case):
    """(cached, new) tokens of every request of a step: ragged histories, or equal numbers of new tokens behind them."""
    n = case["requests"]
    new = lengths(n, case["new"], case["spread"] if not case["cached"] else 0.0, hi=4 * case["new"])
    cached = lengths(n, case["cached"], case["spread"], hi=4 * case["cached"]) if case["cached"] else [0] * n
    return list(zip(cached, new))


def loop_lengths(case):
    """Histories of the returning and of the new users of one turn."""
    lo, hi = case["mean"] // 4, 4 * case["mean"]
    back = [max(s, case["new"] + 1) for s in lengths(case["returning"], case["mean"], 0.6, lo, hi)]
    return back, lengths(case["requests"] - case["returning"], case["mean"], 0.6, lo, hi)


def lookup_bytes(case, n, bag):
    row = case["d"] * esize(case)
    return n * 8 + min(n, case["rows"] * case.get("tables", 1)) * row + n // bag * row


def step_work(case, reqs):
    L, d, e = case["L"], case["d"], esize(case)
    n = sum(t for _, t in reqs)
    pairs = sum(t * p + t * (t + 1) // 2 for p, t in reqs)
    kv = sum(p + t for p, t in reqs) * 2 * L * d * e  # cached keys and values read, new ones written
    return {"bytes": lookup_bytes(case, n * case["bag"], case["bag"]) + n * d * e + kv + 5 * L * d * d * e,
            "flops": L * (10 * d * d * n + 4 * d * pairs)}


def work(case):
    kind = case["kind"]
    if kind == "step":
        return step_work(case, step_lengths(case))
    if kind == "loop":
        back, fresh = loop_lengths(case)
        return step_work(case, [(s - case["new"], case["new"]) for s in back] + [(0, s) for s in fresh])
    if kind == "lookup":
        return {"bytes": lookup_bytes(case, case["lookups"], case["bag"]) + (case["lookups"] if case["flags"] else 0), "flops": 0}
    if kind == "tables":
        n = case["tables"] * case["tokens"]
        return {"bytes": lookup_bytes(case, n, case["bag"]) + 4 * n, "flops": 0}
    row = case["d"] * esize(case)
    removed = (case["high"] - case["low"]) * case["pages"] * 512
    return {"bytes": lookup_bytes(case, case["lookups"], 1) + 4 * removed * row + 8 * case["rows"], "flops": 0}


def tolerance(case):
    if case["kind"] not in ("step", "loop"):
        return "exact"  # rows, flags and the cache's contents
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    # scores, keys, values and outputs are rounded to eight bits in every layer
    return {"rel": 1e-2, "max": 0.15}


# ---- inputs -----------------------------------------------------------------------------------------------------------
class State:
    turn = 0


def generator(seed, stream):
    g = torch.Generator(device=D.DEV)
    g.manual_seed(seed * 1000 + stream)
    return g


def zipf_ids(gen, rows, s, n):
    """n row numbers with P(rank) ~ rank^-s, ranks scattered over the rows by a fixed bijection."""
    u = torch.rand(n, generator=gen, device=D.DEV, dtype=torch.float64)
    top = rows + 1.0
    x = top ** u if abs(s - 1.0) < 1e-9 else (u * (top ** (1.0 - s) - 1.0) + 1.0) ** (1.0 / (1.0 - s))
    return scatter(x.long().clamp_(1, rows) - 1, rows)


def scatter(ranks, rows):
    a = int(rows * 0.6180339887) | 1
    while math.gcd(a, rows) != 1:
        a += 2
    return (ranks * a + 12345) % rows


def feature_ids(gen, case, n):
    """Ids of n output rows: with pooling, feature f of a row draws from a row range of its own."""
    bag, rows = case["bag"], case["rows"]
    if bag == 1:
        return zipf_ids(gen, rows, case["zipf"], n)
    per = rows // bag
    return torch.stack([zipf_ids(gen, per, case["zipf"], n) + f * per for f in range(bag)], dim=1).reshape(-1)


def make_table(seed, rows, d, dtype):
    """A pinned host table."""
    if dtype == "fp32":
        t = torch.empty((rows, d), dtype=torch.float32, pin_memory=True)
        t.copy_(torch.randn((rows, d), generator=generator(seed, 90), device=D.DEV))
        return t
    t = torch.empty((rows, d), dtype=torch.int16, pin_memory=True)
    synth.fill_table_bf16_torch(t, seed, D.DEV)
    return t.view(torch.bfloat16)


def make_timelines(gen, length):
    """Non-decreasing timestamps in seconds, [TIMELINES][length]: lognormal gaps with a median of a minute."""
    gaps = torch.exp(torch.randn((TIMELINES, length), generator=gen, device=D.DEV) * 1.5 + math.log(60.0)).long()
    return 1_600_000_000 + torch.cumsum(gaps, dim=1)


def elem_of(case):
    return B.ELEM_F32 if case["dtype"] == "fp32" else B.ELEM_BF16


def fill_cache(pool, rows):
    """Every row of the table(s) enters the hot cache, as far as its sets have room."""
    for lo in range(0, rows, REFILL_CHUNK):
        ids = torch.arange(lo, min(rows, lo + REFILL_CHUNK), dtype=torch.int64, device=D.DEV)
        check(B.emb_refill(pool.h, ids))


def check(rc):
    if rc not in (B.OK, B.DEFERRED):
        raise RuntimeError("%d %s" % (rc, B.last_error()))


def round_pages(n):
    return (int(n) // 32 + 1) * 32


def make_model(case, seed, n_pos):
    w = synth.make_weights(np.random.default_rng(seed), case["L"], case["d"], case["H"], n_pos, N_TIME, case["dtype"] == "bf16")
    return D.Model(case["L"], case["d"], case["H"], elem_of(case), case["page_tokens"], n_pos, N_TIME, float(n_pos), w)


def make_step_pool(s, case, seed, kv_pages):
    """A pool with kv_pages or a few more pages on the KV side and a hot cache with room for the table twice over."""
    page = s.model.page_size()
    row = case["d"] * esize(case)
    emb_pages = 2 * case["rows"] * row // page + 32
    n_pages = round_pages(emb_pages + kv_pages)
    s.table = make_table(seed, case["rows"], case["d"], case["dtype"])
    s.pool = D.Pool(n_pages, page, row, elem_of(case), case["page_tokens"], 32, s.table, emb_pages / n_pages, zero_fill=True)
    s.first_kv = s.pool.stats()["pages_emb"]
    s.kv = s.pool.mem.view(D.torch_dtype(elem_of(case)))[s.first_kv * page // esize(case):]
    gen = generator(seed, 91)
    for piece in s.kv.split(1 << 28):  # cached keys and values
        piece.normal_(0.0, 0.35, generator=gen)


def prepare_step(case, seed):
    s, rng, gen = State(), np.random.default_rng(seed), generator(seed, 0)
    lens = step_lengths(case)
    rng.shuffle(lens)
    pt, longest = case["page_tokens"], max(p + t for p, t in lens)
    reqs, n_pt, n_ts, n = synth.make_requests([p for p, _ in lens], [t for _, t in lens], pt)
    s.model = make_model(case, seed, longest)
    make_step_pool(s, case, seed, n_pt)
    check(B.pool_reserve(s.pool.h, s.model.h, max_lookups=max(n * case["bag"], REFILL_CHUNK), max_requests=len(reqs),
                         max_new_tokens=n, max_seq_tokens=longest))
    fill_cache(s.pool, case["rows"])
    # the pages of a request lie scattered over the KV side
    s.pages = torch.from_numpy((s.first_kv + rng.permutation(s.pool.n_pages - s.first_kv)[:n_pt]).astype(np.int32)).to(D.DEV)
    s.ts = make_timelines(gen, longest)
    s.reqs = (B.make_reqs([(p, t, pto, (i % TIMELINES) * longest, xo) for i, (p, t, pto, _, xo) in enumerate(reqs)]), len(reqs))
    s.ids = feature_ids(gen, case, n)
    s.bag = case["bag"]
    s.x = torch.empty((n, case["d"]), dtype=D.torch_dtype(elem_of(case)), device=D.DEV)
    s.y = torch.empty_like(s.x)
    return s


def run_step(s):
    check(B.emb_lookup(s.pool.h, s.ids, s.x, s.bag))
    check(B.hstu_step(s.pool.h, s.model.h, s.reqs, s.pages, s.x, s.ts, s.y))
    return {"x": s.x, "y": s.y, "kv": s.kv}


def prepare_loop(case, seed):
    s, rng, gen = State(), np.random.default_rng(seed), generator(seed, 0)
    s.back, s.fresh = loop_lengths(case)
    rng.shuffle(s.back)
    rng.shuffle(s.fresh)
    s.pt, s.new, s.longest = case["page_tokens"], case["new"], 4 * case["mean"]
    s.model = make_model(case, seed, s.longest)
    make_step_pool(s, case, seed, case["kv_pages"])
    s.n = case["returning"] * s.new + sum(s.fresh)
    s.bag, s.d = case["bag"], case["d"]
    check(B.pool_reserve(s.pool.h, s.model.h, max_lookups=max(s.n * s.bag, REFILL_CHUNK), max_requests=case["requests"],
                         max_new_tokens=s.n, max_seq_tokens=s.longest))
    fill_cache(s.pool, case["rows"])
    # users who will not be seen again fill the KV side, then those who keep coming back are cached
    s.next_key, used = 1 << 20, 0
    s.hot = 4 * case["returning"]
    while used < s.pool.n_pages - s.first_kv:
        tokens = s.fresh[s.next_key % len(s.fresh)]
        check(B.kv_seq_reserve(s.pool.h, s.next_key, tokens)[0])
        used += -(-tokens // s.pt)
        s.next_key += 1
    for user in range(s.hot):
        check(B.kv_seq_reserve(s.pool.h, user, s.back[user % len(s.back)])[0])
    s.ts = make_timelines(gen, s.longest)
    s.id_sets = [feature_ids(gen, case, s.n) for _ in range(3)]
    s.order = rng.permutation(case["requests"]).tolist()
    return s


def run_loop(s):
    turn = s.turn
    s.turn += 1
    n_back, n_fresh = len(s.back), len(s.fresh)
    users = [((turn * n_back + i) % s.hot, s.back[i]) for i in range(n_back)]
    users += [(s.next_key + i, s.fresh[i]) for i in range(n_fresh)]
    s.next_key += n_fresh
    pool = s.pool.h
    reqs, tables, page_off, rows = [], [], 0, 0
    for k in s.order:
        user, tokens = users[k]
        rc, have, _ = B.kv_seq_lookup(pool, user)
        cached = tokens - s.new if rc == B.OK and have >= tokens else 0
        rc, pages = B.kv_seq_reserve(pool, user, tokens)
        check(rc)
        B.kv_seq_pin(pool, user)
        reqs.append((cached, tokens - cached, page_off, (user % TIMELINES) * s.longest, rows))
        tables.append(pages)
        page_off += len(pages)
        rows += tokens - cached
    page_tables = torch.from_numpy(np.concatenate(tables)).pin_memory().to(D.DEV, non_blocking=True)
    ids = s.id_sets[turn % len(s.id_sets)][: rows * s.bag]
    x = torch.empty((rows, s.d), dtype=torch.bfloat16, device=D.DEV)
    y = torch.empty_like(x)
    check(B.emb_lookup(pool, ids, x, s.bag))
    check(B.hstu_step(pool, s.model.h, reqs, page_tables, x, s.ts, y))
    for user, _ in users:
        B.kv_seq_unpin(pool, user)
    return {"x": x, "y": y, "pages": page_tables}


def make_lookup_pool(s, case, rows, frac, room):
    page = 64 * 2 * 4 * case["d"] * esize(case)
    row = case["d"] * esize(case)
    n_pages = round_pages(max(32, room * rows * row / page / frac))
    s.pool = D.Pool(n_pages, page, row, elem_of(case), 64, 32, s.table, frac, zero_fill=True)
    s.slab = s.pool.mem.view(torch.int64)


def prepare_lookup(case, seed):
    s, gen = State(), generator(seed, 0)
    n, bag, rows = case["lookups"], case["bag"], case["rows"]
    s.table = make_table(seed, rows, case["d"], case["dtype"])
    make_lookup_pool(s, case, rows, 0.8, case["room"])
    chunk = min(REFILL_CHUNK, rows)
    check(B.pool_reserve(s.pool.h, None, max_lookups=max(n, chunk)))
    if case["room"] >= 1.0:
        fill_cache(s.pool, rows)
        sets = 4
    else:
        # the hottest rows are in; the batches of a cycle touch several times what the cache holds
        for lo in range(0, int(rows * case["room"]), chunk):
            ranks = torch.arange(lo, min(rows, lo + chunk), dtype=torch.int64, device=D.DEV)
            check(B.emb_refill(s.pool.h, scatter(ranks, rows)))
        sets = max(4, min(256, 4 * rows // n))
    s.id_sets = [feature_ids(gen, case, n // bag) for _ in range(sets)]
    s.bag = bag
    s.call = B.emb_lookup_noalloc if case["call"] == "noalloc" else B.emb_lookup
    s.out = torch.empty((n // bag, case["d"]), dtype=D.torch_dtype(elem_of(case)), device=D.DEV)
    s.hit = torch.empty(n, dtype=torch.uint8, device=D.DEV) if case["flags"] else None
    return s


def run_lookup(s):
    ids = s.id_sets[s.turn % len(s.id_sets)]
    s.turn += 1
    check(s.call(s.pool.h, ids, s.out, s.bag, s.hit))
    return {"rows": s.out, "hit": s.hit, "slab": s.slab}


def prepare_tables(case, seed):
    s, gen = State(), generator(seed, 0)
    T, tokens, rows, d = case["tables"], case["tokens"], case["rows"], case["d"]
    s.table = make_table(seed, rows, d, case["dtype"])
    s.more = [make_table(seed + 7919 * k, rows, d >> (k % 3), case["dtype"]) for k in range(1, T)]
    make_lookup_pool(s, case, rows * T, 0.8, 1.6)
    for t in s.more:
        check(B.pool_add_table(s.pool.h, t, rows, t.shape[1] * 2)[0])
    check(B.pool_reserve(s.pool.h, None, max_lookups=max(T * tokens, REFILL_CHUNK)))
    fill_cache(s.pool, rows * T)
    s.table_of = torch.arange(T, dtype=torch.int32, device=D.DEV).repeat(tokens)
    s.id_sets = [zipf_ids(gen, rows, case["zipf"], T * tokens) for _ in range(2)]
    s.bag = case["bag"]
    s.out = torch.empty((T * tokens // s.bag, d), dtype=torch.bfloat16, device=D.DEV)
    return s


def run_tables(s):
    ids = s.id_sets[s.turn % len(s.id_sets)]
    s.turn += 1
    check(B.emb_lookup_tables(s.pool.h, s.table_of, ids, s.out, s.bag))
    return {"rows": s.out}


def prepare_split(case, seed):
    s, gen = State(), generator(seed, 0)
    rows, n, d = case["rows"], case["lookups"], case["d"]
    s.table = make_table(seed, rows, d, case["dtype"])
    s.low, s.high = case["low"], case["high"]
    s.pool = D.Pool(case["pages"], 64 * 2 * 4 * d * 2, d * 2, B.ELEM_BF16, 64, 32, s.table, s.high, zero_fill=True)
    s.slab = s.pool.mem.view(torch.int64)
    check(B.pool_reserve(s.pool.h, None, max_lookups=max(n, rows)))
    s.ranked = scatter(torch.arange(rows, dtype=torch.int64, device=D.DEV), rows)  # every row, hottest first
    check(B.emb_refill(s.pool.h, s.ranked))
    s.id_sets = [zipf_ids(gen, rows, case["zipf"], n) for _ in range(8)]
    s.out = torch.empty((n, d), dtype=torch.bfloat16, device=D.DEV)
    s.hit = torch.empty(n, dtype=torch.uint8, device=D.DEV)
    return s


def run_split(s):
    ids = s.id_sets[s.turn % len(s.id_sets)]
    s.turn += 1
    rc, low = B.pool_set_split(s.pool.h, s.low)
    check(rc)
    check(B.emb_lookup(s.pool.h, ids, s.out, 1, s.hit))
    rc, high = B.pool_set_split(s.pool.h, s.high)
    check(rc)
    check(B.emb_refill(s.pool.h, s.ranked))
    return {"achieved": [low, high], "rows": s.out, "hit": s.hit, "slab": s.slab}


KINDS = {"step": (prepare_step, run_step), "loop": (prepare_loop, run_loop), "lookup": (prepare_lookup, run_lookup),
         "tables": (prepare_tables, run_tables), "split": (prepare_split, run_split)}


def prepare(case, seed):
    make, run_one = KINDS[case["kind"]]
    s = make(case, seed)
    s.run = run_one
    return s


def run(state):
    return state.run(state)
