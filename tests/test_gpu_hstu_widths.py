"""GPU parity of hstu_step over model widths: fp32 models whose heads are not a multiple of four or 16 wide and whose rows do
not fill a wavefront or a block, bf16 models whose layer halves are fused (64 .. 512) and not (192, 320, above 512)."""
import numpy as np
import pytest

from tests.test_gpu_hstu import Case, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16,d,H,pt", [
    (False, 16, 1, 4), (False, 48, 16, 8), (False, 48, 3, 5), (False, 128, 2, 16), (False, 1024, 16, 16),
    (True, 64, 1, 16), (True, 192, 3, 16), (True, 256, 4, 16), (True, 512, 8, 16),
])
def test_two_steps_with_ragged_lengths(bf16, d, H, pt):
    two_steps(Case(21, 2, d, H, pt, bf16, 100, 16, 160.0, 128), [1, 15, 0, 33, 70], [16, 3, 17, 1, 90])


@pytest.mark.parametrize("d,pt", [(192, 64), (192, 24), (320, 64), (576, 64), (1024, 16)])
def test_separate_layernorm_and_gemm_kernels(d, pt):
    """Widths without fused layer halves: several row tiles of 128 per request, a step of several row blocks of the output
    product, rows of more than 512 elements (two chunks per lane), runs of eight tokens of V whole and across pages."""
    two_steps(Case(23, 1, d, d // 64, pt, True, 600, 16, 600.0, 256), [300, 129, 64, 1, 515], [70, 1, 130, 64, 0])


def two_steps(c, first, more):
    d, bf16 = c.d, c.bf16
    reqs, pts, ts, x = c.inputs([0] * len(first), [a + b for a, b in zip(first, more)])
    o1, o2 = np.concatenate([[0], np.cumsum(first)]), np.concatenate([[0], np.cumsum(more)])
    one = [(0, a, r[2], r[3], int(o)) for a, r, o in zip(first, reqs, o1)]
    two = [(a, b, r[2], r[3], int(o)) for a, b, r, o in zip(first, more, reqs, o2)]
    xa = np.concatenate([x[r[4]: r[4] + a] for a, r in zip(first, reqs)])
    xb = np.concatenate([x[r[4] + a: r[4] + a + b] for a, b, r in zip(first, more, reqs)])
    assert_close(c.run_gpu(one, pts, ts, xa), c.run_oracle(one, pts, ts, xa), bf16, "width %d, step 1" % d)
    assert_close(c.run_gpu(two, pts, ts, xb), c.run_oracle(two, pts, ts, xb), bf16, "width %d, step 2" % d)
    assert c.pool.stats()["bad_pages"] == 0
    c.close()


@pytest.mark.parametrize("d,rounds,rest", [(64, 131072, 1), (256, 131072, 5000), (512, 32768, 130), (512, 32768, 31000)])
def test_more_rows_than_one_round_of_blocks(d, rounds, rest):
    """Whole rounds of row tiles keep their columns together, the rest is cut: every copy of one request gets the same rows."""
    T = 64
    n = (rounds + rest + T - 1) // T
    new = [T] * n
    new[-1] = rounds + rest - T * (n - 1)
    c = Case(22, 1, d, d // 64, 16, True, 100, 16, 64.0, (n * 6 + 31) // 32 * 32)
    reqs, pts, ts, x = c.inputs([0] * n, new)
    for r in reqs:
        ts[r[3]:r[3] + r[1]] = ts[:r[1]]
        x[r[4]:r[4] + r[1]] = x[:r[1]]
    got = c.run_gpu(reqs, pts, ts, x)
    ref = c.run_oracle(reqs[:1], pts, ts, x[:T])
    assert_close(got[:T], ref, True, "first copy")
    for r in reqs[1:]:
        assert np.array_equal(got[r[4]:r[4] + r[1]], got[:r[1]]), r
    c.close()
