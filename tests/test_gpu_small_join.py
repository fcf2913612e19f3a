"""A join of up to 4,096 records is sorted and segmented in one block.  Its rows
must equal, in order, those of the radix passes (taken when a digit width is
asked for): one record a side to 4,097 records, key widths around the digits,
carried values and record ids, packed composite keys, semi-joined records, one
hot key, negative keys, the key of all ones."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu
CASES = [  # left rows, right rows, key values, left and right value columns
    (1, 1, 1, 1, 1), (1, 2, 2, 0, 0), (63, 2, 9, 1, 0), (64, 64, 1, 1, 1), (65, 1000, 255, 2, 1), (1000, 800, 256, 1, 1),
    (1000, 800, 257, 2, 2), (2048, 2048, 1, 1, 1), (2048, 2048, 65_535, 1, 2), (4095, 1, 3, 0, 1), (1, 4095, 1, 1, 0),
    (2000, 2096, 65_537, 1, 1), (2000, 2097, 70_000, 1, 1), (1500, 1500, 1 << 24, 3, 1), (500, 3000, (1 << 31) - 1, 1, 1)]


def both_ways(sess, left, right, key=0):
    out = []
    for rb in (0, 8):
        sess.set_tuning(rb, 0)
        t = sess.join(left, right, key)
        out.append((t.nrows, [sess.column(t, c).clone() for c in range(t.ncols)], sess.stats().segments,
                    sess.stats().path))
        sess.free(t)
    (n, got, ns, p), (m, want, ms, q) = out
    assert n == m and ns == ms and p == q and all(torch.equal(x, y) for x, y in zip(got, want))
    return n


@pytest.mark.parametrize("mode", ["plain", "bound", "negative", "semi", "composite"])
@pytest.mark.parametrize("nl,nr,card,lv,rv", CASES)
def test_rows(sess, nl, nr, card, lv, rv, mode):
    announce(f"small join {nl}+{nr} card={card} values {lv},{rv} {mode}")
    g = torch.Generator().manual_seed(nl * 5 + nr + card)
    lk, rk = (torch.randint(0, card, (n,), generator=g) for n in (nl, nr))
    rk[-1] = lk[0] = card - 1
    if mode == "negative":
        lk, rk = lk - (1 << 31), rk - (1 << 31)
    lk, rk = lk.to(torch.int32).cuda(), rk.to(torch.int32).cuda()
    vals = lambda n, k, at: [torch.arange(n, dtype=torch.int32, device="cuda") * 7 + at + c for c in range(k)]
    kmax = card - 1 if mode == "bound" else -1
    lcols, lvars, rcols, rvars = [lk, *vals(nl, lv, 0)], [0, *range(10, 10 + lv)], [rk, *vals(nr, rv, 5)], [0, *range(20, 20 + rv)]
    if mode == "composite":
        for cols, names, n in ((lcols, lvars, nl), (rcols, rvars, nr)):
            cols.append((torch.arange(n, device="cuda") % 3).to(torch.int32))
            names.append(1)
    try:
        sess.set_join_options(semijoin=2 if mode == "semi" else 1, merge=1, precount=1)
        n = both_ways(sess, sess.table(lvars, lcols, key_max=kmax), sess.table(rvars, rcols, key_max=kmax))
        assert n >= 1 or mode == "composite"
    finally:
        sess.set_tuning()
        sess.set_join_options()
        sess._keep.clear()
