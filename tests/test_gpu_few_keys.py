"""A planned join whose LEFT side holds few distinct keys is grouped by
counting.  Its rows must be the ones, in the order, that the sort of the same
records gives: at the edges of the digit widths (63/64, 255/256, 511/512,
1,023 keys, and 1,024, which the sort takes), with LEFT keys that have no
partner, none at all, and a RIGHT side without values."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu
P1, P2, P3, CONST = 4_100_001, 4_100_002, 4_100_003, 4_100_004
IDS = 4_000_000
X, Y, Z, W = -1, -2, -3, -4


def store(keys, partners, constant):
    """p1: keys x's, each with one of up to 8 y's; p2: y's fan, so that p1 JOIN
    p2 has more than 2^21 rows; p3: the larger table, with some of the x's."""
    g = torch.Generator().manual_seed(keys)
    xs = torch.randperm(IDS, generator=g)[:keys + 1]
    xs[0] = IDS - 1  # the end of the key range
    x = xs.unique()[:keys] if keys > 1 else xs[:1]
    x = x[torch.randperm(keys, generator=g)]
    ys = min(8, keys)
    y = torch.arange(keys) % ys
    fan = (1 << 21) // keys + 97
    w = torch.randint(0, IDS, (ys * fan,), generator=g)
    wy = torch.arange(ys).repeat_interleave(fan)
    n3 = ys * fan + 5000
    x3 = torch.randint(0, IDS, (n3,), generator=g)
    x3 = x3[~torch.isin(x3, x)]
    have = x[:max(1, keys * 2 // 3)] if partners else x[:0]
    x3 = torch.cat([x3, have, have[: have.numel() // 2], torch.arange(n3) % 10 + IDS + 1])[:n3 + 4000]
    z = torch.full_like(x3, CONST) if constant else torch.randint(0, IDS, x3.shape, generator=g)
    s = torch.cat([x, w, x3])
    p = torch.cat([torch.full_like(x, P1), torch.full_like(w, P2), torch.full_like(x3, P3)])
    o = torch.cat([y, wy, z])
    at = torch.randperm(s.numel(), generator=g)
    return [c[at].to(torch.int32).cuda() for c in (s, p, o)]


@pytest.mark.parametrize("keys,partners,constant", [
    (1, True, False), (63, True, True), (64, True, False), (255, True, False), (256, True, False), (511, True, False),
    (512, True, True), (1023, True, False), (1024, True, False), (300, False, False)])
def test_rows(sess, keys, partners, constant):
    announce(f"few keys {keys} partners={partners} constant={constant}")
    sess.load(*store(keys, partners, constant))
    q = [(X, P1, Y), (W, P2, Y), (X, P3, CONST if constant else Z)]
    got = sess.query(q)
    st = sess.stats()
    if partners and keys <= 1023:
        assert st.path == B.MAPSQ_PATH_SEMIJOIN and st.passes == 1 and st.left_rows >= 1 << 21
    sess.set_join_options(semijoin=1)
    try:
        want = sess.query(q)
    finally:
        sess.set_join_options()
    assert sess.stats().path == B.MAPSQ_PATH_SORT and sess.stats().out_rows == st.out_rows
    assert got.nrows == want.nrows and (got.nrows > 0) == partners and got.ncols == want.ncols
    assert list(got.var)[:got.ncols] == list(want.var)[:want.ncols] and got.sorted_col == want.sorted_col
    for c in range(got.ncols):
        assert torch.equal(sess.column(got, c), sess.column(want, c))
    sess.free(got)
    sess.free(want)
