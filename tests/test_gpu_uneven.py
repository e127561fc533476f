"""Uneven look-ups must not cost much more than even ones: one row that most
look-ups name, or one table that holds most of them.  Each test compares times
of two calls on the same card, taken from graph replays; the limits leave room
for noise and lie well below what these calls cost while a long segment or a
long table was one block's chain of loads (given with each).  Results are
checked by the parity tests."""
import pytest
import torch

import paper_2005_04680_amd as pk
from gpu_util import DEV, log, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def graph_us(fn, n=10, rounds=7):
    """Fastest of `rounds` replays of n calls, us per call."""
    fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(n):
            fn()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(rounds):
        e0.record()
        g.replay()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1e3 / n)
    return best


class Call:
    """One call's buffers: `bags` look-ups per bag of each table, uniform over its rows, a share
    `hot` of them of row 0; with `cut` the bags are cut at random (a few of them long)."""

    def __init__(self, rows, batch, bags, dim, hot=0.0, cut=False):
        T = len(rows)
        g = torch.Generator(device=DEV)
        g.manual_seed(1)
        sizes = torch.tensor(bags, device=DEV).repeat_interleave(batch)
        offsets = torch.zeros(T * batch + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(sizes, 0, out=offsets[1:])
        if cut:
            for t, p in enumerate(bags):
                o = offsets[t * batch:(t + 1) * batch + 1]
                at = torch.rand(batch - 1, device=DEV, generator=g).sort()[0]
                o[1:-1] = o[0] + (at * (batch * p)).long()
        idx = []
        for m, p in zip(rows, bags):
            r = torch.randint(0, m, (batch * p,), dtype=torch.int32, device=DEV, generator=g)
            if hot > 0:
                r[torch.rand(r.shape, device=DEV, generator=g) < hot] = 0
            idx.append(r)
        self.batch, self.dim, self.I, self.O = batch, dim, torch.cat(idx), offsets.int()
        self.ns = self.I.numel()
        self.tables = pk.Tables([torch.zeros(m, dim, device=DEV) for m in rows])
        self.status = torch.zeros(1, dtype=torch.int32, device=DEV)
        self.ws = torch.empty(pk.embbag_backward_workspace_bytes(T, batch, self.ns, dim),
                              dtype=torch.uint8, device=DEV)
        self.act = torch.ones(T, batch, dim, device=DEV)

    def prepare(self):
        return pk.embbag_backward_prepare(self.tables, self.dim, self.batch, self.I, self.O, self.ws,
                                          self.status)

    def apply(self):
        return pk.embbag_backward_apply_sgd(self.act, self.batch, self.ns, 1e-3, self.tables, self.ws)

    def forward(self):
        return pk.embbag_forward(self.tables, self.batch, self.I, self.O, self.act, self.status)

    def us(self, what):
        assert self.prepare() == 0 and getattr(self, what)() == 0
        t = graph_us(getattr(self, what))
        assert pk.embbag_status_read(self.status) == 0
        return t


# (one fix-up block's chain of loads: 3.1, 2.1 and 1.5 times the even call)
@pytest.mark.parametrize("dim,limit", [(128, 1.9), (256, 1.3), (512, 0.9)])
def test_update_of_one_row(dim, limit):
    even, one = (Call([100_000], 12_500, [40], dim, hot).us("apply") for hot in (0.0, 1.0))
    log(f"[uneven] update E={dim} 500K look-ups: many rows {even:.1f} us, one row {one:.1f} us")
    assert one <= limit * even


# (read one by one, the sums of 256 row groups: 2.5 times the wider rows')
def test_update_of_narrow_rows():
    narrow, wide = (Call([100_000], 1250, [40], dim, 1.0).us("apply") for dim in (4, 32))
    log(f"[uneven] update of one row, 50K look-ups: E=4 {narrow:.1f} us, E=32 {wide:.1f} us")
    assert narrow <= 1.9 * wide


def test_prepare_with_few_long_bags():
    """One table of 641 bags of 296 look-ups on average, some of them 1500, among tables of one
    look-up per bag: the bags of a tile are few of its table's, and long (3.0 times the even call
    when each was one thread's loop)."""
    long, even = (Call([1_000_000] * 26, 641, bags, 16, cut=True).us("prepare")
                  for bags in ([296] + [1] * 25, [12] * 26))
    log(f"[uneven] prepare of 200K look-ups over 26 tables: long bags {long:.1f} us, even {even:.1f} us")
    assert long <= 2.1 * even


# (96K: 2.7 times the even call by tiles merged, 1.3 by table.  The others: 2.0, 1.64
# and 2.35 where the counts were read in words of two, by tiles of at most 4096; 1.46,
# 1.29 and 1.26 now.  The limits lie between.)
@pytest.mark.parametrize("batch,long,each,limit", [(512, 180, 23, 1.9), (4096, 120, 16, 1.72), (8192, 120, 16, 1.55),
                                                   (16384, 115, 15, 1.75)])
def test_prepare_of_one_long_table(batch, long, each, limit):
    """Most look-ups in one of 8 tables, against the same number shared by all: a block of the
    scatter reads the counts of its table's tiles."""
    one, even = (Call([1_000_000] + [100] * 7, batch, bags, 16).us("prepare")
                 for bags in ([long] + [1] * 7, [each] * 8))
    log(f"[uneven] prepare of {batch * (long + 7)} look-ups over 8 tables: one long {one:.1f} us, even {even:.1f} us")
    assert one <= limit * even


# (1.54 times the even call where the walk of a group was 16 look-ups on average, as long
# as the even one now)
def test_forward_of_one_long_table():
    one, even = (Call([100_000] * 26, 2048, bags, 256).us("forward")
                 for bags in ([100] + [1] * 25, [5] * 26))
    log(f"[uneven] forward over 26 tables, E=256: one long {one:.1f} us, even {even:.1f} us")
    assert one <= 1.3 * even
