"""GPU: values that are infinite or not numbers reach the tokens that see them and no earlier ones, in fp32 models, whose attention
multiplies whole tiles of 16 keys and 16 queries."""
import numpy as np
import pytest
import torch

from paper_2605_04450_amd import binding as B
from paper_2605_04450_amd import device as Hn
from tests.test_gpu_hstu import Case

pytestmark = pytest.mark.gpu
WIDTHS = [(64, 4, 16), (64, 2, 16), (96, 2, 6), (64, 1, 4), (80, 5, 5)]  # heads of 16, 32, 48, 64 and 16 elements


@pytest.mark.parametrize("d,H,pt", WIDTHS)
@pytest.mark.parametrize("prefix", [0, 21])
def test_earlier_tokens_do_not_see_a_token_that_is_not_a_number(d, H, pt, prefix):
    c = Case(31, 2, d, H, pt, False, 64, 16, 64.0, 64)
    new, odd_at = [40, 17, 1, 33], [9, 16, 0, 31]
    reqs, pts, ts, x = c.inputs([0] * 4, [prefix + n for n in new])
    if prefix:
        first = [(0, prefix, r[2], r[3], prefix * i) for i, r in enumerate(reqs)]
        c.run_gpu(first, pts, ts, np.concatenate([x[r[4]:r[4] + prefix] for r in reqs]))
    offs = np.concatenate([[0], np.cumsum(new)])
    step = [(prefix, n, r[2], r[3], int(o)) for n, r, o in zip(new, reqs, offs)]
    xs = np.concatenate([x[r[4] + prefix:r[4] + prefix + n] for n, r in zip(new, reqs)])
    want = c.run_gpu(step, pts, ts, xs)
    for o, t in zip(offs, odd_at):
        xs[o + t] = np.nan
    got = c.run_gpu(step, pts, ts, xs)
    for o, n, t in zip(offs, new, odd_at):
        assert np.array_equal(got[o:o + t], want[o:o + t])
        assert np.isnan(got[o + t:o + n]).all()
    c.close()


@pytest.mark.parametrize("d,H,pt", WIDTHS)
def test_an_infinite_value_stays_in_its_element_and_behind_its_token(d, H, pt):
    n = 50
    c = Case(32, 1, d, H, pt, False, 64, 16, 64.0, 64)
    reqs, pts, ts, x = c.inputs([0], [n])
    c.run_gpu(reqs, pts, ts, x)  # keys and values of all tokens
    q = torch.from_numpy(np.random.default_rng(5).standard_normal((n, d)).astype(np.float32)).to(Hn.DEV)
    pages, ts_d = torch.from_numpy(pts).to(Hn.DEV), torch.from_numpy(ts).to(Hn.DEV)

    def attend():
        o = torch.empty_like(q)
        assert B.hstu_attn_paged(c.pool.h, c.model.h, 0, reqs, pages, q, ts_d, o) == B.OK
        return o.cpu().numpy()

    want = attend()
    for token, head, elem, value in ((0, 0, 3, np.inf), (13, H - 1, d // H - 1, -np.inf), (37, 0, 5, np.nan), (49, 0, 0, np.inf)):
        at = Hn.kv_block_elem_offset(1, d, H, pt, int(pts[token // pt]), 0, 1, head) + elem * pt + token % pt
        before = float(c.mem[at])
        c.mem[at] = value
        got = attend()
        c.mem[at] = before
        col = head * (d // H) + elem
        keep = np.ones_like(got, dtype=bool)
        keep[token:, col] = False
        assert np.array_equal(got[keep], want[keep])
        assert (np.isnan(got[token:, col]) if np.isnan(value) else np.isinf(got[token:, col])).all()
    assert np.array_equal(attend(), want)
    c.close()
