"""GPU parity of the miss path and of the refill at batch sizes around whole stretches of the lists and around the sizes of
their grids, with few and with many new ids per set."""
import numpy as np
import pytest

from paper_2605_04450_amd import synth
from tests.test_gpu_emb import check_state, make_pair, run_batches
from tests import test_gpu_emb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,bag,n", [
    (64, 1, 63), (64, 1, 64), (64, 1, 65),                    # one stretch of 64 lookups, and one more
    (64, 1, 512 * 64), (64, 1, 512 * 64 + 1),                 # 512 whole stretches, and one more
    (64, 4, 512 * 128), (64, 4, 512 * 128 + 4),               # pooled: stretches of 128
    (32, 3, 3 * 43691), (32, 16, 16 * 17),                    # the kernel for any row width and bag
])
def test_batches_around_the_borders_of_the_miss_path(d, bag, n):
    rng = np.random.default_rng(n + d)
    rows = 40000
    table = rng.standard_normal((rows, d)).astype(np.float32)
    pool, orc = make_pair(128, 64 * d * 4, d, False, 16, 32, table, 0.5)  # 4096 slots: evictions and bypasses
    cold = rng.integers(0, rows, size=n).astype(np.int64)
    few = np.where(rng.random(n) < 0.01, rng.integers(0, rows, size=n), cold[0]).astype(np.int64)  # long runs of one id
    run_batches(pool, orc, table, [cold, few, synth.zipf_ids(rng, rows, 1.0, n)], bag=bag, tag="border")
    pool.close()


@pytest.mark.parametrize("sets,w_max,frac", [(1, 32, 1.0), (2, 32, 0.5), (3, 32, 1.0), (5, 16, 0.75), (7, 1, 1.0), (64, 32, 0.25)])
def test_new_ids_of_one_set_around_its_number_of_ways(sets, w_max, frac):
    # a batch brings 0, 1, a few or more new ids than ways to a set, next to hits, empty ways and ids seen twice
    rng = np.random.default_rng(sets * 100 + w_max)
    rows, d = 20000, 12  # rows of 48 bytes: fewer 16-byte pieces than lanes
    table = rng.standard_normal((rows, d)).astype(np.float32)
    pool, orc = make_pair(w_max, sets * d * 4, d, False, 16, w_max, table, frac)
    batches = []
    for n in (1, 2, 3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 200, 1000, 5000):
        for share in (1.0, 0.3):  # of ids not seen before, mostly
            seen = np.concatenate(batches)[-100:] if batches else np.arange(4)
            batches.append(np.where(rng.random(n) < share, rng.integers(0, rows, size=n), rng.choice(seen, size=n)).astype(np.int64))
    run_batches(pool, orc, table, batches, tag="new ids of one set")
    for n in (1, 33, 700):
        test_gpu_emb.refill_both(pool, orc, rng.integers(0, rows, size=n), rows)
        check_state(pool, orc, table, "refill")
        run_batches(pool, orc, table, [rng.integers(0, rows, size=n)], tag="after a refill")
    pool.close()


@pytest.mark.parametrize("w_max,n", [(32, 127), (32, 129), (32, 8193 * 128), (8, 1000)])
def test_refills_around_whole_stretches(w_max, n):
    rng = np.random.default_rng(n)
    rows, d = 300000, 8
    table = rng.standard_normal((rows, d)).astype(np.float32)
    pool, orc = make_pair(128, 256 * d * 4, d, False, 16, w_max, table, 0.75)
    for _ in range(2):  # the second one finds most of its ids resident or their sets full
        test_gpu_emb.refill_both(pool, orc, rng.integers(-3, rows + 5, size=n), rows)
        check_state(pool, orc, table, "refill")
    pool.close()
