"""The key sample that decides on the exact pre-count, by what it decides: the
profile shows whether the exact count ran.  Keys from 0, negative keys and keys
far from 0, bounds known or not; few values (whose counters share a line),
hot keys that are sampled, sorted sides, and more sampled keys to a block than
its table holds."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu
N = (1 << 23) + 77
COUNT = 2  # the phase of the sample, the exact count and the count after the sort


def sampled(k):
    return ((k >> 6) * 0x9E3779B1 & 0xFFFFFFFF) >> 26 == k & 63


HOT = next(k for k in range(9000, 20_000) if sampled(k))


def random(seed, hi, n=N):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(0, hi, (n,), generator=g, device="cuda", dtype=torch.int32)


def with_hot(a, rows):
    a[:: a.numel() // rows] = HOT
    return a


def few(rows):
    """60 values of its own, but for `rows` rows"""
    a = random(2, 60) + 10_000
    a[:rows] = random(3, 700, rows)
    return a


def joined(sess, a, b, known, precount):
    """(rows, matching rows checked, count-phase intervals)"""
    va = torch.arange(a.numel(), dtype=torch.int32, device="cuda")
    vb = torch.arange(b.numel(), dtype=torch.int32, device="cuda")
    top = int(max(a.max(), b.max())) if known else -1
    sess.set_join_options(semijoin=1, merge=1, precount=precount)
    B.mapsq_profile_enable(sess.ctx, True)
    try:
        t = sess.join(sess.table([0, 1], [a, va], key_max=top), sess.table([0, 2], [b, vb], key_max=top), 0)
        n = t.nrows
        if 0 < n < 1 << 27:
            k, x, y = (sess.column(t, c) for c in range(3))
            assert torch.equal(a[x.long()], k) and torch.equal(b[y.long()], k)
        sess.free(t)
        return n, B.mapsq_profile_read(sess.ctx).launches[COUNT]
    finally:
        B.mapsq_profile_enable(sess.ctx, False)
        sess.set_join_options()
        sess._keep.clear()


CASES = {  # left, right, whether the sample is followed by the exact count
    "spread": lambda: (random(1, 1 << 22), random(2, 1 << 22), False),
    "wide": lambda: (random(1, 1 << 26), random(2, 1 << 26), False),
    "few_values": lambda: (random(1, 700), few(20_000), False),
    "few_values_many_rows": lambda: (random(1, 700), few(100_000), True),
    "few_against_many": lambda: (random(1, 1000, 1 << 24), random(2, 1000, 5000), False),
    "hot": lambda: (with_hot(random(1, 1 << 23), 1000), with_hot(random(2, 1 << 23), 1000), False),
    "very_hot": lambda: (with_hot(random(1, 1 << 23), 40_000), with_hot(random(2, 1 << 23), 40_000), True),
    "sorted": lambda: (random(1, 1 << 21).sort().values, random(2, 1 << 21).sort().values, False),
    "evens_and_odds": lambda: (random(1, 1 << 22) * 2, random(2, 1 << 22) * 2 + 1, True),
}


@pytest.mark.parametrize("base,known", [(0, True), (0, False), (-(1 << 31), False), (-5_000_001, False),
                                        (1_900_000_000, False)])
@pytest.mark.parametrize("name", list(CASES))
def test_decision(sess, name, base, known):
    announce(f"pre-count sample: {name}, keys from {base}")
    a, b, exact = CASES[name]()
    span = int(max(a.max(), b.max())) + 1
    want = int((torch.bincount(a, minlength=span) * torch.bincount(b, minlength=span)).sum())
    a, b = a + base, b + base
    rows, without = joined(sess, a, b, known, 1)
    assert rows == want
    rows, intervals = joined(sess, a, b, known, 0)
    assert rows == want
    if want == 0:
        assert intervals == 2  # the sample and the exact count; nothing is sorted
    else:
        assert intervals == without + (2 if exact else 1)
