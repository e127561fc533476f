"""GPU parity of the update's segmented reduce where segments meet the edges of
row groups' chunks and of blocks: a segment inside a block is completed from
the block's partial sums in LDS, one that crosses blocks by the fix-up from
the blocks' partial sums.  Tolerance: the update's, |gpu - oracle| <= 1e-6 +
1e-5 |oracle| (the sums are FP64 on both sides).
"""
import numpy as np
import pytest

from gpu_util import GpuTables, require_gpu
from layout_util import lanes as _lanes, layout
from test_gpu_parity import _tables, check_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _check(lengths, dim, split, rng, what):
    M = len(lengths) + 3
    look = np.repeat(np.arange(len(lengths)) + 1, lengths).astype(np.int32)
    rng.shuffle(look)
    batch = look.size // 19 + 1
    cuts = np.sort(rng.integers(0, look.size + 1, batch - 1))
    O = np.concatenate([[0], cuts, [look.size]]).astype(np.int32)
    G = rng.standard_normal((1, batch, dim)).astype(np.float32)
    check_step(_tables(rng, (M,), dim, 0.01), batch, look, O, G, 0.1, split=split, what=what)


# look-ups that a block walks at these sizes: 8 per row group (32 where a row
# takes a whole wavefront), 256 / lanes row groups
@pytest.mark.parametrize("dim,split", [(4, False), (8, True), (16, False), (20, True), (64, False),
                                       (100, False), (128, True), (256, False), (512, True),
                                       (768, False), (1024, False)])
def test_segments_around_chunks_and_blocks(dim, split):
    lanes = _lanes(dim)
    c, groups = (32 if lanes == 64 else 8), 256 // lanes
    span = c * groups
    rng = np.random.default_rng(dim)
    # a span of one-look-up segments first, so that long ones start anywhere
    kinds = [1, 2, c - 1, c, c + 1, 2 * c + 1, span - 1, span, span + 1, 2 * span, 3 * span + c]
    lengths = rng.permutation(np.repeat(kinds, [40, 20, 9, 9, 9, 9, 2, 2, 2, 1, 1]))
    _check(lengths, dim, split, rng, f"blocks of {span} E={dim}")


@pytest.mark.parametrize("dim,split,extra", [(4, False, 0), (8, True, 1), (16, False, -1), (64, False, 0),
                                             (128, True, -1), (256, False, 1), (512, True, 0),
                                             (768, False, 1), (1024, False, -1)])
def test_segment_over_many_blocks(dim, split, extra):
    """A segment over more blocks than the fix-up looks at in one step (64, then a
    search), and segments over about as many as a boundary's own row groups add (4,
    2 or 1 each); all end at, before or after a block's edge."""
    lanes = _lanes(dim)
    groups = 256 // lanes
    span = (32 if lanes == 64 else 8) * groups
    own = groups * {1: 4, 2: 2}.get(-(-dim // 256), 1)
    _check(np.array([span - 3, 258 * span + 3 + extra, 5, (groups + 2) * span + 1, own * span - 1,
                     own * span, own * span + 1, (own + 1) * span + 2]), dim, split,
           np.random.default_rng(dim), f"long segment E={dim}")


@pytest.mark.parametrize("dim,blocks,lead", [(128, 4098, 0), (128, 4098, 15)] + [
    (dim, blocks, lead) for dim, blocks in ((256, 2050), (512, 1026), (1024, 1040))
    for lead in (0, 1, 14, 15, 16, 33)])
def test_groups_of_blocks_are_presummed(dim, blocks, lead):
    """Calls whose partial sums may be over 4 MB: one segment fills groups of 16
    blocks, beginning and ending at every kind of place in its first and last group."""
    span = 256 * 8 if dim == 128 else 128
    lengths = [lead * span + 7] if lead else []
    tail = {0: 40, 1: 16 * 3 + 1, 14: 31, 15: 32, 16: 20, 33: 100}[lead]
    rest = blocks * span - sum(lengths) - tail * span
    _check(np.array(lengths + [tail * span - 5, rest // 3, rest - rest // 3 - 3, 1]), dim, dim == 512,
           np.random.default_rng(lead), f"presummed groups E={dim} lead={lead}")


@pytest.mark.parametrize("dim,ns,chunk", [(64, 150_000, 12), (64, 300_000, 20), (128, 80_000, 12),
                                          (128, 150_000, 20), (32, 1_100_000, 12), (256, 600_000, 40),
                                          (64, 2_500_000, 40), (64, 3_300_000, 52)])
def test_segments_around_other_chunks(dim, ns, chunk):
    """Chunks that are no power of two."""
    L = layout(1, ns // 19 + 1, ns, dim, 200_000)
    assert L.chunk == chunk
    groups = 256 // _lanes(dim)
    span = chunk * groups
    rng = np.random.default_rng(ns)
    kinds = [1, 2, chunk - 1, chunk, chunk + 1, 2 * chunk + 1, span - 1, span, span + 1, 3 * span + 5]
    lengths = rng.choice(kinds, 2 * ns // 20, p=[0.3, 0.1] + [0.13] * 4 + [0.02] * 4)
    lengths = lengths[:int(np.searchsorted(np.cumsum(lengths), ns))]
    _check(np.r_[lengths, ns - lengths.sum()], dim, False, rng, f"chunks of {chunk} E={dim}")


@pytest.mark.parametrize("dim,split", [(4, False), (16, True), (64, False), (256, False), (512, False)])
def test_infinities_and_nan_stay_in_their_rows(dim, split):
    """A gradient of infinity or NaN reaches the rows that its bag names and no other, whichever way
    their sums take: inside a chunk, through a block or over blocks."""
    lanes = _lanes(dim)
    span = (32 if lanes == 64 else 8) * (256 // lanes)
    rng = np.random.default_rng(dim)
    lengths = rng.permutation(np.r_[np.ones(60, int), rng.integers(2, 30, 40), [span + 3, 5 * span, 40 * span, 2]])
    M = len(lengths) + 2
    look = np.repeat(np.arange(len(lengths)), lengths).astype(np.int32)
    rng.shuffle(look)
    batch = look.size // 3
    O = np.r_[np.arange(batch) * 3, look.size].astype(np.int32)
    G = rng.standard_normal((1, batch, dim)).astype(np.float32)
    W = [rng.uniform(-1, 1, (M, dim)).astype(np.float32)]
    bad = rng.choice(batch, 4, replace=False)
    G[0, bad, dim // 2] = [np.inf, -np.inf, np.nan, np.inf]
    gt = GpuTables(W, split=split)
    assert gt.backward(G, batch, look, O, 0.1) == 0 and gt.read_status() == 0
    bag = np.minimum(np.arange(look.size) // 3, batch - 1)
    acc = np.zeros((M, dim))
    np.add.at(acc, look, G[0].astype(np.float64)[bag])
    touched = np.zeros(M, bool)
    touched[look] = True
    with np.errstate(invalid="ignore"):
        ref = np.where(touched[:, None], W[0] - np.float64(np.float32(0.1)) * acc, W[0])
    got = gt.host()[0]
    if split:  # (the halves of a NaN: any NaN, an infinity's low half is zero)
        assert np.array_equal(np.isfinite(got), np.isfinite(ref))
    else:
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    fin = np.isfinite(ref)
    assert np.abs(got[fin] - ref[fin]).max() <= 1e-6 + 1e-5 * np.abs(ref[fin]).max()
    assert 0 < (~fin).sum() <= 4 * 3 + 4


@pytest.mark.parametrize("ns", [1, 7, 8, 9, 127, 128, 129, 255, 256, 257])
def test_last_block(ns):
    """The last block holds any number of look-ups, from one (E = 64: blocks of 128)."""
    rng = np.random.default_rng(ns)
    _check(np.full(1, ns), 64, False, rng, f"one segment of {ns}")
    _check(np.ones(ns, int), 64, True, rng, f"{ns} segments")
