"""GPU parity of the paged attention at the edges of its tiles: query tiles of up to 64 queries (paired wavefronts), of 65
and more, sequences that end inside a 16-byte run of keys, pages smaller than a key tile and not a power of two, items of one
and of several key tiles."""
import numpy as np
import pytest
import torch

from paper_2605_04450_amd import binding as B
from paper_2605_04450_amd import device as Hn
from paper_2605_04450_amd import synth
from tests.test_gpu_hstu import Case, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,pt", [(64, 64), (128, 16), (128, 8), (256, 64), (128, 24), (512, 128)])
@pytest.mark.parametrize("prefix,new", [
    ([0, 0, 0, 0, 0, 0], [1, 31, 32, 33, 63, 64]),
    ([0, 0, 0, 0], [65, 127, 128, 129]),
    ([1, 63, 64, 65, 200], [1, 64, 32, 63, 7]),         # short appends behind cached keys
    ([509, 700, 1003], [64, 65, 3]),                    # several key tiles and items
])
def test_query_and_key_tile_edges(d, pt, prefix, new):
    c = Case(11, 1, d, d // 64, pt, True, 300, 16, 1024.0, 640)
    total = [p + n for p, n in zip(prefix, new)]
    reqs, pts, ts, x = c.inputs([0] * len(new), total)
    # the cached part through a first step, the new part through a second one
    if any(prefix):
        offs = np.concatenate([[0], np.cumsum(prefix)])
        first = [(0, p, r[2], r[3], int(o)) for p, r, o in zip(prefix, reqs, offs)]
        xa = np.concatenate([x[r[4]: r[4] + p] for p, r in zip(prefix, reqs)])
        assert_close(c.run_gpu(first, pts, ts, xa), c.run_oracle(first, pts, ts, xa), True, "cached part")
    offs = np.concatenate([[0], np.cumsum(new)])
    second = [(p, n, r[2], r[3], int(o)) for p, n, r, o in zip(prefix, new, reqs, offs)]
    xb = np.concatenate([x[r[4] + p: r[4] + p + n] for p, n, r in zip(prefix, new, reqs)])
    assert_close(c.run_gpu(second, pts, ts, xb), c.run_oracle(second, pts, ts, xb), True, "new part")
    assert c.pool.stats()["bad_pages"] == 0
    c.close()


@pytest.mark.parametrize("pt", [16, 64])
def test_values_behind_the_end_of_a_sequence_do_not_matter(pt):
    c = Case(12, 1, 128, 2, pt, True, 256, 16, 256.0, 64)
    reqs, pts, ts, x = c.inputs([0, 0], [101, 67])
    c.pool.mem.view(torch.int16).fill_(0x7FC0)  # NaN everywhere
    assert_close(c.run_gpu(reqs, pts, ts, x), c.run_oracle(reqs, pts, ts, x), True, "NaN behind the end")
    c.close()


@pytest.mark.parametrize("pt", [16, 64, 128])
@pytest.mark.parametrize("ordered", [True, False])
def test_items_of_one_to_ten_key_tiles(pt, ordered):
    # so many query tiles that none is cut: their items have 2, 4, 6, 8 and 9 or 10 key tiles, an odd or even last one, one
    # that ends at its 64th key or before; the window's ring of 256 distances wraps twice
    lens = [64 * 10, 64 * 10 - 1, 64 * 9, 64 * 9 - 5, 64 * 8 + 1, 64 * 10 - 32, 64, 65, 129] + [640] * 55
    c = Case(13, 1, 512, 8, pt, True, 300, 24, 640.0, (60000 // pt // 32 + 2) * 32)
    reqs, pts, ts, x = c.inputs([0] * len(lens), lens)
    if not ordered:
        for r in reqs[:9:2]:  # these requests take the general path
            ts[r[3] + r[1] // 2] -= 100_000
    got = c.run_gpu(reqs, pts, ts, x)
    some = reqs[:9]
    n = some[-1][4] + some[-1][1]
    assert_close(got[:n], c.run_oracle(some, pts, ts, x[:n]), True, "items of many key tiles")
    assert c.pool.stats()["bad_pages"] == 0
    c.close()


# (tests/host_san/schedule.cpp holds the numbers of partials and the kernels to these)
@pytest.mark.parametrize("d,n,prefix,new", [
    (64, 40, 1100, 64), (64, 41, 1100, 64),   # the most blocks of attention_reduce_rows, nine partials a tile, and one tile more
    (128, 20, 1100, 61), (128, 21, 1100, 61),  # of two heads, the last block with one row
    (64, 41, 1000, 64), (64, 40, 1000, 64),   # eight partials: attention_reduce
    (64, 64, 520, 64), (128, 33, 600, 1),     # five: a round of four and one more
    (64, 1, 4500, 64), (64, 1, 4000, 64), (64, 1, 1000, 128),  # 36, 32 and 9: two rounds, a full one, part of one
    (64, 64, 200, 64), (256, 1, 300, 3), (256, 1, 200, 2),     # two
])
def test_sums_of_few_and_many_partials(d, n, prefix, new):
    """Requests with the same rows and keys: the first one as the oracle computes it, the others like the first."""
    S = prefix + new
    c = Case(14, 1, d, d // 64, 64, True, 300, 16, 1024.0, (n * -(-S // 64) * 4 // 3 // 32 + 2) * 32)
    reqs, pts, ts, x = c.inputs([0] * n, [S] * n)
    for r in reqs:
        ts[r[3]:r[3] + S] = ts[:S]
        x[r[4]:r[4] + S] = x[:S]
    first = [(0, prefix, r[2], r[3], i * prefix) for i, r in enumerate(reqs)]
    xa = np.concatenate([x[:prefix]] * n)
    c.run_gpu(first, pts, ts, xa)
    c.run_oracle(first[:1], pts, ts, xa[:prefix])
    second = [(prefix, new, r[2], r[3], i * new) for i, r in enumerate(reqs)]
    xb = np.concatenate([x[prefix:S]] * n)
    got = c.run_gpu(second, pts, ts, xb)
    assert_close(got[:new], c.run_oracle(second[:1], pts, ts, xb[:new]), True, "first copy")
    for i in range(1, n):
        assert np.array_equal(got[i * new:(i + 1) * new], got[:new]), i
    c.close()


@pytest.mark.parametrize("d,n,pieces,new", [
    (64, 1, 5, 1), (64, 1, 6, 64), (128, 2, 7, 33), (256, 1, 8, 64), (256, 16, 12, 64),      # attention_reduce, rounds of four
    (64, 1, 9, 64), (64, 2, 16, 3), (256, 1, 17, 64), (256, 1, 24, 64), (512, 1, 32, 128),   # attention_reduce_rows: one round
    (64, 1, 33, 64), (128, 1, 48, 2), (64, 1, 49, 100), (256, 1, 94, 1),                     # and several
])
def test_partials_are_added_in_the_order_of_the_keys(d, n, pieces, new):
    """Pieces of two key tiles, q.k = 1 for every pair and one value other than zero in each piece: M in the first, between a
    quarter and half a unit in M's last place in those that follow, -M in the last.  Added in the order of the keys they leave
    M as it is each time, and then exactly nothing; any two of the small ones added first leave more."""
    S, H = 128 * pieces, d // 64
    w = synth.make_weights(np.random.default_rng(1), 1, d, H, 16, 16, True)
    w["pos"][:] = 0
    w["time"][:] = 0
    model = Hn.Model(1, d, H, B.ELEM_BF16, 64, 16, 16, 1.0, w)
    n_pages = (S // 64 // 32 + 2) * 32
    pool = Hn.Pool(n_pages, model.page_size(), d * 2, B.ELEM_BF16, 64, 32, None, 0.0, zero_fill=True)
    k = torch.zeros((S, d), dtype=torch.bfloat16, device=Hn.DEV)
    v = torch.zeros_like(k)
    k[:, ::64] = 1.0
    big = 1 + torch.arange(d, device=Hn.DEV) % 64 / 128
    v[::128] = (big * 2.0 ** -25).bfloat16()
    v[0], v[S - 128] = big, -big
    pages = np.arange(n_pages - S // 64, n_pages, dtype=np.int32)
    Hn.write_prefix_kv(pool.mem.view(torch.bfloat16), 1, d, H, 64, pages, k, v, 0)
    q = torch.zeros((n * new, d), dtype=torch.bfloat16, device=Hn.DEV)
    q[:, ::64] = 1.0
    o = torch.empty_like(q)
    reqs = [(S - new, new, 0, 0, i * new) for i in range(n)]  # of the same pages
    ts = torch.arange(S, dtype=torch.int64, device=Hn.DEV)
    assert B.hstu_attn_paged(pool.h, model.h, 0, reqs, torch.from_numpy(pages).to(Hn.DEV), q, ts, o) == B.OK
    assert not o.any()
    v[S - 128] = 0  # without the last one: M times SiLU(1), as bf16 has it
    Hn.write_prefix_kv(pool.mem.view(torch.bfloat16), 1, d, H, 64, pages, k, v, 0)
    assert B.hstu_attn_paged(pool.h, model.h, 0, reqs, torch.from_numpy(pages).to(Hn.DEV), q, ts, o) == B.OK
    want = big.double() / (1 + np.exp(-1.0))
    assert ((o.double() - want).abs() <= 2 ** -8 * want * 1.01).all()  # half a unit each: SiLU(1) and the output, in bf16
    model.close()
    pool.close()
