"""GPU parity of steps whose layer halves are joined in one kernel, where its split changes: the number of column slices, the
last group of 32 rows, and the number of rows from which the halves are kernels of their own.  Every request is a copy of the
first one, which the oracle computes, and gets the same rows; two layers, so that a back half feeds a front half."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_04450_amd import device as Hn
from paper_2605_04450_amd import synth
from tests.test_gpu_hstu import Case, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,rows", [
    (64, 1), (64, 31), (64, 4096), (64, 4097), (64, 65536), (64, 65537),
    (128, 33), (128, 2048), (128, 2081), (128, 8192), (128, 65536), (128, 65537),
    (256, 32), (256, 1024), (256, 1025), (256, 4097), (256, 8191), (256, 24576), (256, 24577),
    (512, 65), (512, 512), (512, 513), (512, 2049), (512, 8192), (512, 8193),
    # the last rows of a number of slices and the first of the next
    (64, 8160), (64, 8161),
    (128, 4064), (128, 4065), (128, 8160), (128, 8161),
    (256, 2016), (256, 2017), (256, 4064), (256, 4065), (256, 8160), (256, 8161),
    (512, 1024), (512, 1025), (512, 2048), (512, 4096), (512, 4097),
])
def test_copies_of_one_request_get_the_same_rows(d, rows):
    T = min(rows, 37)
    n = (rows + T - 1) // T
    new = [T] * n
    new[-1] = rows - T * (n - 1)
    c = Case(24, 2, d, d // 64, 24, True, 100, 16, 64.0, (n * 4 + 31) // 32 * 32 + 32)
    reqs, pts, ts, x = c.inputs([0] * n, new)
    for r in reqs:
        ts[r[3]:r[3] + r[1]] = ts[:r[1]]
        x[r[4]:r[4] + r[1]] = x[:r[1]]
    got = c.run_gpu(reqs, pts, ts, x)
    assert_close(got[:T], c.run_oracle(reqs[:1], pts, ts, x[:T]), True, "first copy")
    for r in reqs[1:]:
        assert np.array_equal(got[r[4]:r[4] + r[1]], got[:r[1]]), r
    assert c.pool.stats()["bad_pages"] == 0
    c.close()


@pytest.mark.parametrize("d,new", [(64, 2067), (128, 300), (256, 33), (512, 64)])
def test_the_first_layers_kernel_looks_at_every_timestamp(d, new):
    """Its blocks take 2048 tokens of a request each: a decrease at either end of these is counted and computed as such."""
    c = Case(25, 1, d, d // 64, 24, True, 100, 16, 64.0, 160)
    reqs, pts, ts, x = c.inputs([0, 0], [new, 5])
    assert_close(c.run_gpu(reqs, pts, ts, x), c.run_oracle(reqs, pts, ts, x), True, "ordered")
    assert c.pool.stats()["unordered_ts"] == 0
    at = [j for j in (1, 2047, 2048, 2049) if j < new - 1] + [new - 1]
    for n, j in enumerate(at):
        t = ts.copy()
        t[j] = t[j - 1] - 1
        got = c.run_gpu(reqs, pts, t, x)
        assert c.pool.stats()["unordered_ts"] == n + 1, j
        if n == 0 or j == at[-1]:
            assert_close(got, c.run_oracle(reqs, pts, t, x), True, "decrease at %d" % j)
    c.close()


# (d = 64, one head, is below, behind cached keys: the attention of a request's first token is then SiLU(q.k) v / n of a single key, whose relative error has
# no bound where q.k, a sum of terms rounded to eight bits, is near zero, and the second LayerNorm takes the scale away.  Of several
# heads not all are near zero at once.)
@pytest.mark.parametrize("d,T", [(128, 3), (256, 1), (256, 15), (256, 16), (512, 11)])
def test_rows_of_many_requests_in_a_group(d, T):
    # a group of 32 rows holds rows of one, two or more requests; each finds the pages of its own
    n = 70
    c = Case(26, 2, d, d // 64, 8, True, 100, 16, 64.0, 800)
    reqs, pts, ts, x = c.inputs([0] * n, [T + (i % 3 == 0) for i in range(n)])
    assert_close(c.run_gpu(reqs, pts, ts, x), c.run_oracle(reqs, pts, ts, x), True, "short requests")
    bad = pts.copy()
    bad[reqs[40][2]] = c.pool.n_pages + 3  # a page that is not there: counted, and nobody else's rows change
    got, ref = c.run_gpu(reqs, bad, ts, x), c.run_oracle(reqs, pts, ts, x)
    keep = np.ones(len(x), bool)
    keep[reqs[40][4]: reqs[40][4] + reqs[40][1]] = False
    assert_close(got[keep], ref[keep], True, "beside a bad page")
    assert c.pool.stats()["bad_pages"] > 0
    c.close()


@pytest.mark.parametrize("d,T", [(64, 1), (64, 3), (64, 11), (64, 16), (128, 3)])
def test_rows_of_many_requests_in_a_group_behind_cached_keys(d, T):
    n, P = 70, 21
    c = Case(27, 2, d, d // 64, 8, True, 100, 16, 64.0, 608)
    new = [T + (i % 3 == 0) for i in range(n)]
    whole, pts, ts, _ = c.inputs([P] * n, new)
    x = synth.as_bf16_values(c.rng.standard_normal((sum(new), d)).astype(np.float32))
    for (_, _, pto, _, _) in whole:
        pages = pts[pto:pto + -(-P // 8)]
        for layer in range(2):
            k, v = (synth.as_bf16_values(c.rng.standard_normal((P, d)).astype(np.float32)) for _ in range(2))
            Hn.write_prefix_kv(c.mem, 2, d, c.H, 8, pages, torch.from_numpy(k).to(Hn.DEV).bfloat16(), torch.from_numpy(v).to(Hn.DEV).bfloat16(), layer)
            for j in range(P):
                for h in range(c.H):
                    for which, rows in enumerate((k, v)):
                        at = oracle.kv_offset(c.cfg, int(pages[j // 8]), layer, which, h, j % 8)
                        c.kv[at:at + 64] = rows[j, 64 * h:64 * h + 64]
    assert_close(c.run_gpu(whole, pts, ts, x), c.run_oracle(whole, pts, ts, x), True, "short appends")
    assert c.pool.stats()["bad_pages"] == 0
    c.close()
