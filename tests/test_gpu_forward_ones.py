"""Forward of bags that hold one look-up each (copied) or nearly so: pooled
outputs must be the oracle's bits, whatever the width, storage and pooling, at
the edges of the groups of bags that a row group takes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2005_04680_amd as pk
from gpu_util import DEV, GpuTables, bf16_bits, bits_equal, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _bags(T, batch, kind, rng):
    sizes = np.ones(T * batch, int)
    if kind == "two and none":  # one look-up on average, not in every bag
        sizes[3::11] = 2
        sizes[5::11] = 0
    elif kind == "first long":
        sizes[0] = 40
    O = np.r_[0, np.cumsum(sizes)].astype(np.int32)
    return O


@pytest.mark.parametrize("kind", ["one", "two and none", "first long"])
@pytest.mark.parametrize("dim,batch", [(4, 5), (8, 300), (16, 17), (20, 4096), (64, 1), (64, 2047),
                                       (128, 16), (128, 4001), (256, 33), (512, 5), (1024, 130)])
def test_pooled_bits(dim, batch, kind):
    rng = np.random.default_rng(dim + batch)
    rows = (7, 4000, 1)
    O = _bags(3, batch, kind, rng)
    I = np.concatenate([rng.integers(0, m, O[(t + 1) * batch] - O[t * batch])
                        for t, m in enumerate(rows)]).astype(np.int32)
    W = [rng.standard_normal((m, dim)).astype(np.float32) for m in rows]
    W[0][3] = -0.0
    W[1][7::9] *= np.float32(1e-42)  # subnormal and tiny rows
    print(dim, batch, kind, flush=True)
    gt = GpuTables(W)
    rc, Y = gt.forward(batch, I, O)
    assert rc == 0 and gt.read_status() == 0
    assert bits_equal(Y.cpu().numpy(), oracle.forward(W, batch, I, O)[1])
    Id, Od = to_dev(I), to_dev(O)
    a = rng.uniform(-2, 2, I.size).astype(np.float32)
    for w, mode, om in ((a, pk.EMBBAG_POOL_SUM, oracle.POOL_SUM),
                        (None, pk.EMBBAG_POOL_MEAN, oracle.POOL_MEAN)):
        assert pk.embbag_forward_pooled(gt.w, batch, Id, Od, Y, None if w is None else to_dev(w),
                                        mode, gt.status) == 0
        assert bits_equal(Y.cpu().numpy(), oracle.forward_weighted(W, batch, I, O, w, om)[1])
    gs = GpuTables(W, split=True)
    his = [oracle.split(w)[0] for w in W]
    rc, Y = gs.forward(batch, I, O)
    assert rc == 0
    assert bits_equal(Y.cpu().numpy(), oracle.forward_split(his, batch, I, O)[1])
    Yb = torch.empty((3, batch, dim), dtype=torch.bfloat16, device=DEV)
    assert pk.embbag_forward_split_bf16_act(gs.w, batch, Id, Od, Yb, gs.status) == 0
    assert bits_equal(bf16_bits(Yb), oracle.forward_split_bf16_act(his, batch, I, O)[1])
    assert gs.read_status() == 0


@pytest.mark.parametrize("dim,T,batch,avg", [(256, 26, 1300, 2), (256, 26, 1300, 3), (256, 26, 1301, 4),
                                             (256, 33, 1299, 7), (64, 12, 11003, 4), (20, 40, 8000, 3)])
@pytest.mark.parametrize("kind", ["even", "ragged", "one long table"])
def test_pooled_bits_of_short_groups(dim, T, batch, avg, kind):
    """Grids large enough for groups of several bags whose tables have few groups."""
    rng = np.random.default_rng(dim + avg)
    sizes = np.full((T, batch), avg)
    if kind == "ragged":
        sizes = rng.integers(0, 2 * avg + 1, (T, batch))
    elif kind == "one long table":
        sizes[:] = 1
        sizes[T // 2] = T * (avg - 1) + rng.integers(0, 3, batch)
    O = np.r_[0, np.cumsum(sizes.ravel())].astype(np.int32)
    I = rng.integers(0, 900, O[-1]).astype(np.int32)
    W = [rng.standard_normal((900, dim)).astype(np.float32) for _ in range(T)]
    print(dim, T, batch, avg, kind, I.size, flush=True)
    gt = GpuTables(W)
    rc, Y = gt.forward(batch, I, O)
    assert rc == 0 and gt.read_status() == 0
    assert bits_equal(Y.cpu().numpy(), oracle.forward(W, batch, I, O)[1])


@pytest.mark.parametrize("dim", [16, 64, 256])
def test_infinities_and_nan_are_copied(dim):
    """A row's infinities and NaN reach the bags that name it and no other."""
    rng = np.random.default_rng(dim)
    W = [rng.standard_normal((50, dim)).astype(np.float32) for _ in range(3)]
    W[0][3], W[1][4], W[2][5, 1] = np.inf, np.nan, -np.inf
    batch = 3000
    O = np.arange(3 * batch + 1, dtype=np.int32)
    I = rng.integers(0, 50, 3 * batch).astype(np.int32)
    a = rng.uniform(-2, 2, I.size).astype(np.float32)
    gt = GpuTables(W)
    rc, Y = gt.forward(batch, I, O)
    ref = np.stack([W[t][I[t * batch:(t + 1) * batch]] for t in range(3)])
    assert rc == 0 and np.array_equal(Y.cpu().numpy(), ref, equal_nan=True)
    assert pk.embbag_forward_pooled(gt.w, batch, to_dev(I), to_dev(O), Y, to_dev(a),
                                    pk.EMBBAG_POOL_SUM, gt.status) == 0
    ref = (ref.astype(np.float64) * a.reshape(3, batch, 1)).astype(np.float32)
    assert np.array_equal(Y.cpu().numpy(), ref, equal_nan=True)
    assert gt.read_status() == 0


@pytest.mark.parametrize("bad", [7, -1])
def test_index_out_of_range(bad):
    O = np.arange(3 * 700 + 1, dtype=np.int32)
    I = np.zeros(2100, np.int32)
    I[1399] = bad
    gt = GpuTables([np.ones((7, 128), np.float32)] * 3)
    rc, _ = gt.forward(700, I, O)
    assert rc == 0 and gt.read_status() == pk.EMBBAG_ERR_INDEX_RANGE


@pytest.mark.parametrize("dim", [32, 128, 512])
@pytest.mark.parametrize("shift,bad_at", [(1, 3), (0, -4)])
def test_bad_offsets_win_over_a_bad_index(dim, shift, bad_at):
    """One look-up in every bag, but the list starts at 1 (or ends before
    num_indices), and a group of bags that sees this also reads a bad index."""
    T, batch = 3, 700
    O = np.arange(T * batch + 1, dtype=np.int32) + shift
    I = np.zeros(T * batch + 1, np.int32)  # one look-up more than the bags hold
    I[bad_at] = 7
    gt = GpuTables([np.ones((7, dim), np.float32)] * T)
    rc, _ = gt.forward(batch, I, O)
    assert rc == 0 and gt.read_status() == pk.EMBBAG_ERR_OFFSETS
