"""Radix passes of 9 to 11 bits, where a block has more digits than threads: the
rows are those of 8-bit passes, in order, for whole tiles and remainders, one
tile and many, spread and hot digits, keys that end inside the last digit, one
join at a time and batched."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu


def side(g, n, bits, hot, lo):
    a = torch.randint(0, 1 << bits, (n,), generator=g, device="cuda", dtype=torch.int64)
    if hot:  # most records in the first and the last digit of every pass
        a = torch.where(torch.rand(n, generator=g, device="cuda") < 0.6, (a & 1) * ((1 << bits) - 1), a)
    a[-1] = (1 << bits) - 1
    return (a + lo).to(torch.int32)


def tables(sess, n, m, bits, hot, values):
    g = torch.Generator(device="cuda").manual_seed(n + bits)
    lo = -(1 << 31) if bits == 32 else 0
    out = []
    for k, first in ((n, 1), (m, 10)):
        a = side(g, k, bits, hot, lo)
        if hot:  # one row a hot key on the smaller side keeps the result small
            a = a if k == n else a.unique()
        cols = [a, *(torch.arange(a.numel(), dtype=torch.int32, device="cuda") + c for c in range(values))]
        out.append(sess.table([0, *range(first, first + values)], cols, key_max=-1))
    return out


@pytest.mark.parametrize("kpt", [8, 16])
@pytest.mark.parametrize("rb", [9, 10, 11])
@pytest.mark.parametrize("n,m,bits,hot,values", [
    (4097, 4095, 20, False, 1), (8192, 8192, 22, False, 2), (60_000, 5_537, 31, False, 1), (70_001, 3_000, 32, False, 1),
    (300_000, 200_001, 24, True, 1), (1_500_000, 700_003, 27, False, 2), (400_000, 1000, 9, True, 0)])
def test_joins(sess, n, m, bits, hot, values, rb, kpt):
    announce(f"wide digits {rb}/{kpt}: {n}+{m} bits={bits} hot={hot} values={values}")
    L, R = tables(sess, n, m, bits, hot, values)
    out = []
    try:
        sess.set_join_options(semijoin=1, merge=1, precount=1)
        for tuning in ((rb, kpt), (8, kpt)):
            sess.set_tuning(*tuning)
            t = sess.join(L, R, 0)
            assert sess.stats().radix_bits == tuning[0]
            out.append([sess.column(t, c).clone() for c in range(t.ncols)])
            sess.free(t)
    finally:
        sess.set_tuning()
        sess.set_join_options()
        sess._keep.clear()
    assert out[0][0].numel() >= 1 and all(torch.equal(x, y) for x, y in zip(*out))


@pytest.mark.parametrize("kpt", [0, 8, 16])
@pytest.mark.parametrize("rb", [9, 10, 11])
def test_batches(sess, rb, kpt):
    announce(f"wide digits {rb}/{kpt}: batch")
    joins = [(*tables(sess, n, m, bits, hot, values), 0) for n, m, bits, hot, values in (
        (1, 1, 3, False, 1), (2048, 2049, 12, False, 1), (8191, 40_000, 20, False, 2), (50_000, 3_000, 31, False, 1),
        (200_000, 90_001, 22, True, 1))]
    try:
        sess.set_tuning(rb, kpt)
        got = sess.join_batch(joins)
        sess.set_tuning(8, 0)
        want = sess.join_batch(joins)
        for a, b in zip(got, want):
            assert a.nrows == b.nrows >= 1
            assert all(torch.equal(sess.column(a, c), sess.column(b, c)) for c in range(a.ncols))
            sess.free(a)
            sess.free(b)
    finally:
        sess.set_tuning()
        sess._keep.clear()
