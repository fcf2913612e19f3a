"""A key bound that does not hold (key_max below the keys): the rows are wrong,
but they are the rows of a definite join, and every kernel stays inside its
arrays.  The keys are cut to the bits of the bound, so the join must equal,
row for row, the join of the cut keys under a bound that holds; the semi-join
drops what lies outside the bound from the larger side.  Sizes around the
segment kernels' tiles, with runs of one key that go on past a tile."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu
HI = 1 << 10


def sides(n, m, negative):
    """keys over four times the bound; every 3rd of a few hot ones, in and out of it"""
    g = torch.Generator(device="cuda").manual_seed(n)
    out = []
    for k in (n, m):
        a = torch.randint(0, 4 * HI, (k,), generator=g, device="cuda", dtype=torch.int32)
        hot = torch.tensor([5, HI + 5, 3 * HI + 9], dtype=torch.int32, device="cuda")
        at = torch.rand(k, generator=g, device="cuda") < 0.3
        a = torch.where(at, hot[torch.randint(0, 3, (k,), generator=g, device="cuda")], a)
        out.append(a - 2 * HI if negative else a)
    return out


def columns(sess, a, b, values):
    def table(k, first):
        return sess.table([0, *range(first, first + values)],
                          [k, *(torch.arange(k.numel(), dtype=torch.int32, device="cuda") + c for c in range(values))],
                          key_max=HI - 1)
    t = sess.join(table(a, 1), table(b, 9), 0)
    got = [sess.column(t, c).clone() for c in range(t.ncols)]
    path = sess.stats().path
    sess.free(t)
    return got, path


@pytest.mark.parametrize("negative", [False, True])
@pytest.mark.parametrize("values", [1, 2])  # carried through the sort, gathered by record id
@pytest.mark.parametrize("n,m", [(900, 700), (5000, 3000), (20_000, 4097), (300_000, 1200)])
def test_the_sorts(sess, n, m, values, negative):
    announce(f"key bound that does not hold: sort {n}+{m} values={values} negative={negative}")
    a, b = sides(n, m, negative)
    try:
        sess.set_join_options(semijoin=1, merge=1, precount=1)
        got, path = columns(sess, a, b, values)
        want, _ = columns(sess, a & (HI - 1), b & (HI - 1), values)
    finally:
        sess.set_join_options()
        sess._keep.clear()
    assert path == B.MAPSQ_PATH_SORT and len(want[0]) > 0
    assert all(torch.equal(x, y) for x, y in zip(got, want))


@pytest.mark.parametrize("n,m", [(900, 700), (20_000, 4097), (300_000, 1200)])
def test_the_semi_join(sess, n, m):
    announce(f"key bound that does not hold: semi-join {n}+{m}")
    a, b = sides(n, m, False)
    kept = (a < HI) & torch.isin(a, b[b < HI])  # of the larger side
    try:
        sess.set_join_options(semijoin=2, merge=1, precount=1)
        got, path = columns(sess, a, b, 1)
        sess.set_join_options(semijoin=1, merge=1, precount=1)
        want, _ = columns(sess, a[kept], b & (HI - 1), 1)
    finally:
        sess.set_join_options()
        sess._keep.clear()
    want[1] = torch.nonzero(kept).flatten().to(torch.int32)[want[1].long()]
    assert path == B.MAPSQ_PATH_SEMIJOIN and len(want[0]) > 0
    assert all(torch.equal(x, y) for x, y in zip(got, want))
