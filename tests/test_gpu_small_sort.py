"""Small calls sort tile by tile in LDS, mid-sized ones table by table: the sorted (key, bag) words, unique
keys and segment offsets must be those of a stable sort, bit for bit, at the
edges of tiles (2048 or 4096 look-ups of a table), of the one-block form (4096 in all)
and of the path's range; data errors are reported as by the radix sort.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2005_04680_amd as pk
from gpu_util import DEV, GpuTables, assert_close, gpu_dedup, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _batch(rng, rows, batch, counts, hot=0.0):
    """Look-ups with counts[t] of them in table t, over its `batch` bags at random."""
    O = [0]
    I = []
    for m, n in zip(rows, counts):
        cuts = np.sort(rng.integers(0, n + 1, batch - 1))
        O += list(O[-1] + np.r_[cuts, n])
        r = rng.integers(0, m, n)
        r[rng.random(n) < hot] = m // 2
        I.append(r)
    return np.concatenate(I).astype(np.int32), np.array(O, np.int32)


def _reference(rows, batch, I, O):
    bag = np.searchsorted(O[1:], np.arange(I.size), side="right").astype(np.uint32)
    base = np.r_[0, np.cumsum(rows)]
    key = (base[bag // batch] + I).astype(np.uint32)
    order = np.argsort(key, kind="stable")
    uniq, first = np.unique(key[order], return_index=True)
    return key[order], bag[order], uniq, np.r_[first, I.size]


CASES = {
    "one look-up": ((7,), 1, (1,)),
    "one row": ((1,), 3, (300,)),
    "one block, full": ((5, 1000), 40, (1096, 3000)),
    "one block, many empty bags": ((100, 100), 15000, (700, 20)),
    "two kernels, nothing to merge": ((5, 1000, 90000), 40, (1097, 3000, 4096)),
    "a tile and one look-up": ((1 << 20, 9), 700, (4097, 1)),
    "empty tables between": ((50, 50, 3000, 50), 64, (0, 9000, 0, 4095)),
    "31 key bits, eight tiles": ((2147483000,), 100, (32768,)),
    "all in one table": ((300000, 10, 10), 500, (98304, 0, 0)),
    "64 tables": (tuple(range(1, 65)), 70, tuple(64 * i for i in range(1, 41)) + (0,) * 24),
    "more bags than a block's threads": ((70000, 800), 9000, (12289, 5000)),
    "last size of the path": ((200000,) * 4, 3000, (30000, 30000, 30000, 8304)),
    "first size past it": ((200000,) * 4, 3000, (30000, 30000, 30000, 8305)),
    "small, tiles of 4096": ((200000, 1 << 21, 300), 800, (27000, 40960, 8193)),
    "by table, 64 tables of 20 bits": ((1 << 20,) * 64, 40, (1536,) * 63 + (1600,)),
    "by table, last of 2048": ((90000, 5, 1 << 20), 20000, (262144, 2049, 260095)),
    "by table, first of 4096": ((90000, 5, 1 << 20), 20000, (262144, 2049, 260096)),
    "by table, one row each": ((1, 1), 700, (60000, 40000)),
    "by table, one pass": ((1000, 3, 1024), 9000, (40960, 4097, 90000)),
    "by table, two passes": ((1 << 20, 700, 5), 50, (0, 100000, 4096)),
    "by table, three passes": ((1 << 20, (1 << 20) + 1), 50000, (99999, 8193)),
    "by table, four passes": ((2147483000,), 3000, (32769,)),
    "by table, 64 tables": ((50000,) * 64, 40, (1,) * 31 + (0,) + (3300,) * 32),
    "by table, last per table": ((300000,), 900, (262144,)),
    "whole list, first per table": ((300000,), 900, (262145,)),
    "few long bags of many": ((30000, 9, 1 << 20), 700, (2100, 699, 200000)),
    "long bags, one block": ((300, 70), 300, (3000, 600)),
    "by table, 32 tiles of a table and 33": ((1 << 20, 1 << 19), 3000, (65536, 65537)),
    "by table, first of 8192": ((1 << 20, 70000, 9, 5), 9000, (1040384, 8192, 1, 0)),
    "by table, 8192 and remainders": ((1 << 20,) * 6, 9000, (8191, 8193, 16384, 900000, 300001, 77)),
    "by table, last of 8192": ((1 << 20, 3, 3, 3, 3, 3, 3, 3), 9000, (2064384, 0, 0, 0, 0, 0, 0, 0)),
    "by table, first past 8192": ((1 << 20, 3, 3, 3, 3, 3, 3, 3), 9000, (2064385, 0, 0, 0, 0, 0, 0, 0)),
    "by table, digits of 3 bits": ((2, 5, 2), 900, (70000, 40000, 3)),
    "tiles, last size": ((200000,) * 4, 3000, (30000, 30000, 1000, 440)),
    "tiles, first size past it": ((200000,) * 4, 3000, (30000, 30000, 1000, 441)),
    "tiles, all in one table": ((300000, 10, 10), 500, (61440, 0, 0)),
    "by table, counts of a narrower digit": ((1000000,) + (100,) * 63, 40, (970,) * 64),
    "by table, the same of 4096 in one": ((1000000,) + (100,) * 63, 40, (62000,) + (7,) * 63),
    "by table, most skewed": ((300000, 5, 5, 5, 5, 5, 5), 900, (1835008, 0, 0, 0, 0, 0, 0)),
}


def test_bags_of_any_length_in_a_tile():
    """Bags of 1 to 5000 look-ups, long ones filled by a wavefront together (more
    than 128 per thread of the bag), among as many empty ones as leave a bag one, two
    or four threads."""
    rng = np.random.default_rng(11)
    for bags, longest in ((300, 600), (600, 130), (600, 1500), (1100, 5000), (5000, 900)):
        sizes = np.where(rng.random(bags) < 0.03, rng.integers(100, longest + 1, bags),
                         rng.integers(0, 2, bags))
        for d in (127, 128, 129, 256, 257, 512, 513):
            sizes[rng.integers(0, bags)] = min(d, longest)
        print(bags, longest, int(sizes.sum()), flush=True)
        O = np.r_[0, np.cumsum(np.r_[sizes, sizes[::-1]])].astype(np.int32)
        I = rng.integers(0, 40000, O[-1]).astype(np.int32)
        rc, status, got = gpu_dedup((40000, 50000), bags, I, O)
        key, bag, uniq, seg = _reference((40000, 50000), bags, I, O)
        assert rc == 0 and status == 0
        assert np.array_equal(got["sorted_keys"], key) and np.array_equal(got["sorted_bags"], bag)


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("hot", [0.0, 0.6])
def test_sorted_as_by_a_stable_sort(name, hot):
    rows, batch, counts = CASES[name]
    rng = np.random.default_rng(len(name))
    I, O = _batch(rng, rows, batch, counts, hot)
    print(name, "NS", I.size, flush=True)
    rc, status, got = gpu_dedup(rows, batch, I, O)
    key, bag, uniq, seg = _reference(rows, batch, I, O)
    assert rc == 0 and status == 0
    assert np.array_equal(got["sorted_keys"], key)
    assert np.array_equal(got["sorted_bags"], bag)
    assert np.array_equal(got["unique_keys"], uniq)
    assert np.array_equal(got["seg_off"], seg)


@pytest.mark.parametrize("counts", [(3000, 1000), (9000, 4000), (70000, 60000),
                                    (400000, 200000)])
def test_data_errors(counts):
    rows, batch = (500, 800), 300
    rng = np.random.default_rng(3)
    I, O = _batch(rng, rows, batch, counts)
    bad_row = I.copy()
    bad_row[counts[0] - 1] = 500
    negative = I.copy()
    negative[0] = -1
    down = O.copy()
    down[17] = down[18] + 5
    short = O.copy()
    short[-1] -= 1
    edge = O.copy()
    edge[batch] = 2 ** 31 - 1
    low, high = O.copy(), O.copy()
    low[batch + 9:batch + 12] = -2 ** 31
    high[20:23] = 2 ** 31 - 1
    for idx, off, code in ((I, low, pk.EMBBAG_ERR_OFFSETS), (I, high, pk.EMBBAG_ERR_OFFSETS),
                           (bad_row, O, pk.EMBBAG_ERR_INDEX_RANGE),
                           (negative, O, pk.EMBBAG_ERR_INDEX_RANGE),
                           (I, down, pk.EMBBAG_ERR_OFFSETS), (I, short, pk.EMBBAG_ERR_OFFSETS),
                           (bad_row, edge, pk.EMBBAG_ERR_OFFSETS)):
        rc, status, _ = gpu_dedup(rows, batch, idx, off)
        assert rc == 0 and status == code
    rc, status, _ = gpu_dedup(rows, batch, I, O)
    assert rc == 0 and status == 0


def test_data_errors_in_large_tiles():
    """The same where tiles hold 8192 look-ups."""
    T, batch, n = 8, 500, 150_000
    rows = (700,) * T
    I, O = _batch(np.random.default_rng(4), rows, batch, (n,) * T)
    bad_row = I.copy()
    bad_row[5 * n + 8192] = 700
    offs = [O.copy() for _ in range(4)]
    offs[0][3 * batch] = -2 ** 31
    offs[1][3 * batch + 7:3 * batch + 9] = 2 ** 31 - 1
    offs[2][-1] -= 1
    offs[3][0] = 1
    rc, status, _ = gpu_dedup(rows, batch, bad_row, O)
    assert rc == 0 and status == pk.EMBBAG_ERR_INDEX_RANGE
    for off in offs:
        rc, status, _ = gpu_dedup(rows, batch, bad_row, off)
        assert rc == 0 and status == pk.EMBBAG_ERR_OFFSETS
    rc, status, _ = gpu_dedup(rows, batch, I, O)
    assert rc == 0 and status == 0


@pytest.mark.parametrize("counts", [(2000, 1500), (9000, 4097), (30000, 4097), (50000, 70000),
                                    (300000, 230000), (490000, 33000)])
def test_weights_travel_with_the_look_ups(counts):
    rows, batch, dim = (900, 40000), 77, 12
    rng = np.random.default_rng(5)
    I, O = _batch(rng, rows, batch, counts, 0.2)
    a = rng.uniform(-2, 2, I.size).astype(np.float32)
    G = rng.standard_normal((2, batch, dim)).astype(np.float32)
    W = [rng.uniform(-0.1, 0.1, (m, dim)).astype(np.float32) for m in rows]
    gt = GpuTables(W)
    ws = torch.empty(pk.embbag_backward_workspace_bytes(2, batch, I.size, dim), dtype=torch.uint8,
                     device=DEV)
    assert pk.embbag_backward_sgd_pooled(to_dev(G), batch, to_dev(I), to_dev(O), 0.1, gt.w, ws,
                                         to_dev(a), pk.EMBBAG_POOL_SUM, gt.status) == 0
    assert gt.read_status() == 0
    assert oracle.backward_sgd_weighted(G, batch, I, O, 0.1, W, a, oracle.POOL_SUM) == 0
    for t, w in enumerate(gt.host()):
        assert_close(w, W[t], f"table {t}")
