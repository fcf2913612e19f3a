"""Batched joins at the edges of their record tiles (2,048, 4,096 and 8,192
records with 8, 16 and 32 keys per thread): segments that end, split or reach
past a tile, one-sided runs, hot keys, filtered and unfiltered joins.  Every
join's rows must equal, in order, those of the same join run alone."""
import pytest
import torch

from tests.conftest import announce

pytestmark = pytest.mark.gpu


def side(g, n, card, hot):
    k = torch.randint(0, card, (n,), generator=g)
    if hot:
        k[torch.rand(n, generator=g) < 0.5] = card // 2
    return k.to(torch.int32).cuda()


@pytest.mark.parametrize("semijoin", [0, 1])
@pytest.mark.parametrize("kpt,tile", [(8, 2048), (16, 4096), (0, 8192)])
def test_rows(sess, kpt, tile, semijoin):
    announce(f"batch tiles kpt={kpt} semijoin={semijoin}")
    g = torch.Generator().manual_seed(tile + semijoin)
    shapes = [(tile // 2, tile // 2, tile, False), (tile - 1, 1, 3, False), (tile, 1, 1, False), (1, tile, 1, False),
              (tile, tile, 40, False), (tile + 1, tile - 1, 100_000, False), (3 * tile, 5, 4, False),
              (7, 2 * tile + 3, 5, False), (63, 64, 9, False), (1, 1, 1, False), (5 * tile, tile // 4, 3 * tile, True),
              (200, 9 * tile + 1, 50, True), (20_000, 30_000, 1 << 20, False), (12 * tile, 11 * tile, 9 * tile, False)]
    joins, keep = [], []
    for i, (nl, nr, card, hot) in enumerate(shapes):
        lk, rk = side(g, nl, card, hot), side(g, nr, card, False)
        rk[0] = lk[-1]
        vals = [torch.arange(n, dtype=torch.int32, device="cuda") + 10 * i for n in (nl, nl, nr)]
        lv, rv = (vals[:1] if i % 3 == 0 else vals[:2]), vals[2:] if i % 4 else []
        joins.append((sess.table([0, 1, 2][: 1 + len(lv)], [lk, *lv], key_max=(1 << 20) - 1),
                      sess.table([0, 3][: 1 + len(rv)], [rk, *rv], key_max=(1 << 20) - 1), 0))
    try:
        sess.set_tuning(0, kpt)
        sess.set_join_options(semijoin=semijoin)
        got = sess.join_batch(joins)
        sess.set_join_options(semijoin=1, precount=1)
        for (left, right, key), t in zip(joins, got):
            want = sess.join(left, right, key)
            assert t.nrows == want.nrows >= 1 and t.ncols == want.ncols
            for c in range(t.ncols):
                assert torch.equal(sess.column(t, c), sess.column(want, c))
            sess.free(t)
            sess.free(want)
    finally:
        sess.set_tuning()
        sess.set_join_options()
        sess._keep.clear()
