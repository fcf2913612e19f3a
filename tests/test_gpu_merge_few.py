"""The merge join at the edges of its small-side search: tiles of 64 keys, the
8,192-row rule, runs on the small side around the 16 rows looked ahead, large
sides of one row to many, keys at the ends of the type.  Rows and their order
must be the shuffle's."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu
LO, HI = -(1 << 31), (1 << 31) - 1


def sides(ns, nb, run, extreme):
    g = torch.Generator().manual_seed(ns * 31 + nb)
    span = max(1, nb // 2)
    heads = torch.randint(0, span, ((ns + run - 1) // run,), generator=g)
    a = heads.repeat_interleave(run)[:ns]
    b = torch.randint(0, span, (nb,), generator=g)
    b[-1] = a[0]
    if extreme:
        a[: ns // 3 + 1], b[: nb // 3 + 1] = LO, LO
        a[-1], b[-1] = HI, HI
    return [x.sort().values.to(torch.int32).cuda() for x in (a, b)]


@pytest.mark.parametrize("ns,nb,run,extreme", [
    (1, 1, 1, False), (1, 70_000, 1, False), (2, 3, 1, True), (63, 64, 1, False), (64, 5000, 16, False),
    (65, 5000, 17, False), (66, 4000, 18, True), (900, 1000, 300, False), (8191, 8192, 1, False),
    (8192, 300_000, 16, False), (8193, 300_000, 17, False), (4000, 1_000_000, 1, False), (300, 2_000_000, 40, True)])
def test_rows(sess, ns, nb, run, extreme):
    announce(f"merge few ns={ns} nb={nb} run={run} extreme={extreme}")
    a, b = sides(ns, nb, run, extreme)
    va, vb = (torch.arange(x.numel(), dtype=torch.int32, device="cuda") for x in (a, b))
    if extreme:  # keep the products small
        b, vb = (torch.cat([x[:2], x[nb // 3 + 1:]]) for x in (b, vb))
    out = []
    try:
        for merge in (0, 1):
            sess.set_join_options(semijoin=1, merge=merge, precount=1)
            for left, right in (((a, va), (b, vb)), ((b, vb), (a, va))):
                t = sess.join(sess.table([0, 1], left, sorted_col=1), sess.table([0, 2], right, sorted_col=1), 0)
                assert sess.stats().path == (B.MAPSQ_PATH_SORT if merge else B.MAPSQ_PATH_MERGE)
                out.append([sess.column(t, c).clone() for c in range(3)])
                sess.free(t)
    finally:
        sess.set_join_options()
        sess._keep.clear()
    for got, want in ((out[0], out[2]), (out[1], out[3])):
        assert got[0].numel() >= 1 and all(torch.equal(x, y) for x, y in zip(got, want))
