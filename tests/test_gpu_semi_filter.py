"""The semi-join's filter at the edges of its mask words, tiles and chunks (a
chunk takes two tiles from 2,048 x 4,096 records on): the join's rows are the
ones, in the order, that the unfiltered sort gives, for keys that repeat, that
ascend (neighbours share a bitmap word) and a few hot ones."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["random", "ascending", "hot"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 4095, 4096, 4097, 12_300, 600_000, 2048 * 4096, 2048 * 4096 + 1,
                               2048 * 8192 + 77])
def test_rows(sess, n, kind):
    announce(f"semi filter n={n} {kind}")
    g = torch.Generator(device="cuda").manual_seed(n)
    m = max(1, n // 9)
    span = 3 * n + 40

    def draw(k):
        a = torch.randint(7, 7 + span, (k,), generator=g, device="cuda", dtype=torch.int32)
        if kind == "hot":
            a = torch.where(torch.rand(k, generator=g, device="cuda") < 0.7, (a % 5) * 3 + 11, a)
        return a.sort().values if kind == "ascending" else a

    big, small = draw(n), draw(m)
    small[-1] = big[-1]  # at least one pair, of the last record
    if kind == "hot":  # keep the result small: one copy of each key on the small side
        small = small.unique()
    vb, vs = (torch.arange(x.numel(), dtype=torch.int32, device="cuda") for x in (big, small))
    out = []
    try:
        for mode in (2, 1):
            sess.set_join_options(semijoin=mode, merge=1, precount=1)
            for left, right in (((big, vb), (small, vs)), ((small, vs), (big, vb))):
                t = sess.join(sess.table([0, 1], left), sess.table([0, 2], right), 0)
                assert sess.stats().path == (B.MAPSQ_PATH_SEMIJOIN if mode == 2 else B.MAPSQ_PATH_SORT)
                out.append([sess.column(t, c).clone() for c in range(3)])
                sess.free(t)
    finally:
        sess.set_join_options()
        sess._keep.clear()
    for got, want in ((out[0], out[2]), (out[1], out[3])):
        assert got[0].numel() >= 1 and all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("at", [1, 2, 63, 64, 65])
def test_a_lone_key_among_neighbours(sess, at):
    """a wave whose keys share one bitmap word but for one, in the lowest word"""
    announce(f"semi filter lone key at {at}")
    small = torch.full((128,), 5000, dtype=torch.int32, device="cuda")
    small[at] = 0
    big = torch.tensor([0, 5000, 4999, 1, 31, 0], dtype=torch.int32, device="cuda").repeat(100)
    try:
        sess.set_join_options(semijoin=2, merge=1, precount=1)
        t = sess.join(sess.table([0], [big]), sess.table([0], [small]), 0)
        assert sess.stats().path == B.MAPSQ_PATH_SEMIJOIN
        assert t.nrows == 200 + 100 * 127
        sess.free(t)
    finally:
        sess.set_join_options()
        sess._keep.clear()
