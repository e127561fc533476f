"""The update's rule for segments that cross row groups and blocks, on the CPU.

The sorted look-ups are cut into chunks of C, one per row group, NG row groups
to a block.  Every segment (the look-ups of one row) is applied once:
  * inside a chunk, or beginning in it and ending at its end, by its row group;
  * beginning in a chunk and going on, by that row group, with the sums that
    the following row groups of the block parked;
  * going on past the block, by the fix-up: the block leaves its part in slot
    2b + 1, the blocks that follow theirs in slot 2b.  A segment over many blocks
    may be added up in aligned groups of 16 of them first, each group's sum in
    the unused slot 2b + 1 of its first block.
A model restates these decisions and is checked on random segment lengths around
those of chunks, blocks and groups; mistakes planted in the model are caught.
The sizes (chunk, blocks, carry slots, room for the sorts' counts) come from the
library's own rule and are checked for every kind of call.  The GPU tests check
the kernels.
"""
import random

import numpy as np
import pytest

from layout_util import lanes, layout

NOKEY = -1
GROUP = 16  # blocks of a pre-summed group


def applied_segments(keys, C, NG, own, Q, presum, wrong=None):
    """Segments as the update applies them: {key: [positions summed]}.  `own`: blocks up to which a
    boundary's own row groups add a segment; Q: boundaries of a fix-up block; `wrong`: a planted
    mistake."""
    NS, span = len(keys), C * NG
    key = lambda i: int(keys[i]) if 0 <= i < NS else NOKEY
    nblk = (NS + span - 1) // span
    carry, out = {}, {}

    def apply(k, pos):
        assert k not in out, f"row {k} applied twice"
        out[k] = pos

    for b in range(nblk):
        parked, thru, last = {}, [False] * NG, {}
        first_open = False
        for g in range(NG):
            lo = (b * NG + g) * C
            hi = min(lo + C, NS) if lo < NS else lo
            if lo >= hi:
                continue
            open_ = key(lo - 1) == key(lo)
            first_open = open_ if g == 0 else first_open
            cur, acc = key(lo), []
            for s in range(lo, hi):
                if key(s) != cur:
                    if open_:
                        parked[g] = acc
                    else:
                        apply(cur, acc)
                    open_, cur, acc = False, key(s), []
                acc.append(s)
            last_open = key(hi) == cur
            thru[g] = open_ and last_open
            if open_:
                parked[g] = acc
            elif not last_open:
                apply(cur, acc)
            else:
                last[g] = (cur, acc)
        if wrong == "chain stops early":
            thru = [False] * NG

        def chain(k):
            got = []
            while k < NG:
                got += parked[k]
                if not thru[k]:
                    return got, False
                k += 1
            return got, True

        for g, (cur, acc) in last.items():
            more, on = chain(g + 1)
            if on:
                carry[2 * b + 1] = acc + more
            else:
                apply(cur, acc + more)
        if first_open:
            carry[2 * b] = chain(0)[0]

    if presum:
        for b0 in range(GROUP, nblk, GROUP):
            if b0 + GROUP < nblk and key(b0 * span - 1) == key((b0 + GROUP) * span):
                assert 2 * b0 + 1 not in carry
                first = 1 if wrong == "group without its first block" else 0
                carry[2 * b0 + 1] = sum((carry[2 * (b0 + u)] for u in range(first, GROUP)), [])

    for base in range(0, nblk - 1, Q):
        long_ones = 0
        for b in range(base, min(base + Q, nblk - 1)):
            lo, hi = b * span, (b + 1) * span
            kl = key(hi - 1)
            if key(hi) != kl or key(lo - 1) == kl:
                continue
            n = 0
            while b + 1 + n < nblk and key((b + 1 + n) * span) == kl:
                n += 1
            slots = [2 * (b + 1 + i) for i in range(n)]
            if n > own:
                long_ones += 1
                g0 = (b + GROUP) // GROUP * GROUP
                groups = (b + n - g0) // GROUP if presum and b + n > g0 else 0
                if wrong == "one group too many" and presum and b + n > g0:
                    groups = (b + n - g0 + GROUP - 1) // GROUP
                if groups > 0:
                    head = g0 - (b + 1)
                    slots = slots[:head] + [2 * (g0 + GROUP * i) + 1 for i in range(groups)] + \
                        slots[head + GROUP * groups:]
            apply(kl, carry[2 * b + 1] + sum((carry[s] for s in slots), []))
        assert long_ones <= 1, "two long segments in one fix-up block"
    return out


def check(lengths, *rule, wrong=None):
    keys = np.repeat(np.arange(len(lengths), dtype=np.int64) * 3 + 1, lengths)
    got = applied_segments(keys, *rule, wrong=wrong)
    starts = np.r_[0, np.cumsum(lengths)]
    assert sorted(got) == [int(k) for k in np.unique(keys)]
    for i, k in enumerate(np.arange(len(lengths)) * 3 + 1):
        assert sorted(got[int(k)]) == list(range(starts[i], starts[i + 1])), f"segment {i} summed wrongly"


# (C, NG, blocks a boundary's own row groups add, boundaries of a fix-up block)
RULES = [(8, 4, 16, 4), (32, 4, 16, 4), (40, 4, 8, 2), (12, 8, 32, 4), (8, 16, 64, 1), (20, 16, 64, 1),
         (52, 16, 64, 1), (12, 32, 128, 1), (8, 256, 1024, 1), (8, 4, 4, 2)]


@pytest.mark.parametrize("rule", RULES)
@pytest.mark.parametrize("presum", [False, True])
def test_every_segment_applied_once(rule, presum):
    C, NG, own, Q = rule
    span = C * NG
    rng = np.random.default_rng(span + own)
    kinds = np.array([1, 2, 3, C - 1, C, C + 1, 2 * C + 1, span - 1, span, span + 1, 2 * span, 3 * span + 5])
    many = np.array([own * span, (own + 1) * span + 1, GROUP * span, 2 * GROUP * span + 1, 40 * span + 3])
    for trial in range(12):
        n = int(rng.integers(1, 40))
        lengths = rng.choice(kinds, n)
        if span <= 700 and own <= 64:
            lengths = rng.permutation(np.r_[lengths, rng.choice(many, 2)])
        elif trial == 0:
            lengths = rng.permutation(np.r_[lengths, 34 * span])
        check(lengths, C, NG, own, Q, presum)


@pytest.mark.parametrize("lead", range(0, 35))
def test_groups_of_blocks_from_every_place(lead):
    span = 32
    for n in (15, 16, 17, 31, 32, 33, 48, 50):
        lengths = [x for x in (lead * span - 3, n * span + 3, 40) if x > 0]
        check(np.array(lengths), 8, 4, 4, 2, True)


@pytest.mark.parametrize("wrong", ["chain stops early", "group without its first block",
                                   "one group too many"])
def test_the_check_sees_planted_mistakes(wrong):
    span = 32
    # (a missing partial sum shows as a KeyError, one taken twice or never as an AssertionError)
    with pytest.raises((AssertionError, KeyError)):
        for lead in range(1, 18):
            for tail in (0, 1, span - 1):
                check(np.array([lead * span - 3, 40 * span + tail, 7, 90]), 8, 4, 4, 2, True, wrong=wrong)


def test_sizes_of_every_call():
    """Chunks cover the list, fit the look-ups in flight and the carry slots; the sorts' counts fit
    their room; a workspace sized without the tables' rows is large enough; positions past the list
    stay below 2^32."""
    rng = random.Random(1)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    edges = [1, 8, 4096, 4097, 32768, 32769, 61440, 61441, 262144, 262145, 524288, 524289, 1048576,
             1048577, 2097152, 2097153, 2 ** 31 - 1]
    for _ in range(40000):
        T = rng.choice([1, 2, 3, 8, 26, 63, 64])
        E = 4 * (log(1, 256) if rng.random() < 0.5 else rng.choice([1, 2, 4, 8, 16, 32, 64, 128, 256]))
        ns = rng.choice(edges) if rng.random() < 0.3 else log(1, 2 ** 31 - 1)
        B = log(1, min((2 ** 31 - 2) // T, 4 * ns // T + 2))
        rows = [log(1, 2 ** 30 // T) for _ in range(T)]
        if rng.random() < 0.3:  # one long table among short ones: wide digits of the whole list
            rows = [log(1, 2 ** 30)] + [rng.randrange(1, 100)] * (T - 1)
        L = layout(T, B, ns, E, sum(rows))
        lpr = lanes(E)
        span = L.chunk * (256 // lpr)
        what = (T, B, ns, E, rows[0])
        assert 8 <= L.chunk <= 256 and L.chunk % (8 if lpr == 64 else 4) == 0, what
        assert (L.nblocks - 1) * span < ns <= L.nblocks * span < 2 ** 32, what
        assert 2 * L.nblocks * E * 8 <= L.off_uniq - L.off_carry, what
        assert L.total <= layout(T, B, ns, E, 0).total, what
        room = L.off_tot - L.off_hist
        bits = max(max(rows) - 1, 1).bit_length()
        tiles = lambda n: -(-ns // n) + T
        assert not (L.small and L.by_table)
        if L.small:
            assert ns <= 15 * 4096 and 28 * tiles(2048) <= room, what
        if L.by_table:
            need = [tiles(4096) * ((2 << max(-(-bits // p), 3)) + 28) for p in range(-(-bits // 10), 5)]
            assert ns <= 512 * 4096 and min(need) <= room, what
