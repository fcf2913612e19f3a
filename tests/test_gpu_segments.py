"""Segments and rows straight from the sorted records at the tile's edges:
segments that end, split or reach past a tile of 1,024 (few records) or 4,096
records (by a few, by more than 64 and by many tiles), one-sided segments there, key products on
both sides of the 64-pair rule, for carried values, record ids and a packed
composite key.  Each result must equal the one the definition gives, row for
row: keys ascending, the side with fewer value bytes inside."""
import numpy as np
import pytest
import torch

from tests.conftest import announce

pytestmark = pytest.mark.gpu
T = 4096  # a multiple of the smaller tile too; `many` lifts a case to the larger one


def rows_of(lk, rk, nlv, nrv):
    """(key, LEFT row, RIGHT row) of every pair in the library's order."""
    lo, ro = np.argsort(lk, kind="stable"), np.argsort(rk, kind="stable")
    ls, rs = lk[lo], rk[ro]
    out = []
    for k in np.intersect1d(ls, rs):
        a = lo[np.searchsorted(ls, k):np.searchsorted(ls, k, "right")]
        b = ro[np.searchsorted(rs, k):np.searchsorted(rs, k, "right")]
        if a.size * nlv < b.size * nrv:  # LEFT inside
            i, j = np.tile(a, b.size), np.repeat(b, a.size)
        else:
            i, j = np.repeat(a, b.size), np.tile(b, a.size)
        out.append(np.stack([np.full(i.size, k), i, j]))
    return np.concatenate(out, 1) if out else np.zeros((3, 0), np.int64)


def counts(name):
    """[(cL, cR)] of keys 0, 1, 2, ..."""
    one = [(1, 1)]
    return {
        "ends_on_the_tile": one * (T // 2) + one * 3,
        "head_is_last_record": one * (T // 2 - 1) + [(1, 0), (1, 1), (2, 3)],
        "split_past_the_tile": one * (T // 2 - 2) + [(4, 2), (1, 1)],
        "ends_60_past": one * (T // 2 - 1) + [(2, 30), (30, 2), (1, 1)],
        "ends_at_64": one * (T // 2 - 2) + [(4, 16), (1, 1)] * 40,
        "one_sided_long": one * (T // 2 - 3) + [(6 + 5000, 0), (1, 1), (0, 9000), (3, 3)],
        "one_sided_then_pairs": one * 700 + [(0, 3 * T)] + one * 900 + [(T, 1)],
        "dense_past_many_tiles": one * 2000 + [(9000, 5), (1, 1), (3, 20_000), (0, 2), (2, 2)],
        "at_64_pairs": [(8, 8), (64, 1), (1, 64), (3, 0), (2, 32)] * 300,
        "over_64_pairs": [(8, 8), (65, 1)] * 200,
        "single_records": [(1, 0), (0, 1)] * 5000 + one,
        "exactly_one_tile": one * (T // 2),
    }[name]


NAMES = ["ends_on_the_tile", "head_is_last_record", "split_past_the_tile", "ends_60_past", "ends_at_64",
         "one_sided_long", "one_sided_then_pairs", "dense_past_many_tiles", "at_64_pairs", "over_64_pairs",
         "single_records", "exactly_one_tile"]


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("values", [(1, 1), (0, 1), (2, 1), (1, 3)])
@pytest.mark.parametrize("name", NAMES)
def test_rows(sess, name, values, many):
    announce(f"segments {name}, {values[0]} + {values[1]} value columns{', many' if many else ''}")
    nlv, nrv = values
    c = np.array(counts(name) + ([(1, 0), (0, 1)] * (1 << 17) if many else []))
    r = np.random.default_rng(5)
    lk = r.permutation(np.repeat(np.arange(len(c)) + 3, c[:, 0])).astype(np.int32)
    rk = r.permutation(np.repeat(np.arange(len(c)) + 3, c[:, 1])).astype(np.int32)
    lv = [r.integers(0, 1 << 30, lk.size).astype(np.int32) for _ in range(nlv)]
    rv = [r.integers(0, 1 << 30, rk.size).astype(np.int32) for _ in range(nrv)]
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    sess.set_join_options(semijoin=1, merge=1, precount=1)
    try:
        L = sess.table([0] + [10 + i for i in range(nlv)], [dev(x) for x in [lk] + lv])
        R = sess.table([0] + [20 + i for i in range(nrv)], [dev(x) for x in [rk] + rv], key_max=len(c) + 3)
        t = sess.join(L, R, 0)
        got = sess.to_numpy(t)
        st = sess.stats()
        sess.free(t)
    finally:
        sess.set_join_options()
        sess._keep.clear()
    k, i, j = rows_of(lk, rk, nlv, nrv)
    assert st.out_rows == k.size and st.segments == int((c.sum(1) > 0).sum())
    want = [k] + [x[i] for x in lv] + [x[j] for x in rv]
    for g, x in zip(got, want):
        assert np.array_equal(g, x)


def test_packed_composite_key(sess):
    """Two shared variables packed in one word: segments of the whole word."""
    announce("segments of a packed composite key")
    r = np.random.default_rng(6)
    n = 3 * T + 5
    cols = [r.integers(0, 40, n).astype(np.int32) for _ in range(4)]
    v = np.arange(n, dtype=np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    L = sess.table([0, 1, 10], [dev(cols[0]), dev(cols[1]), dev(v)])
    R = sess.table([0, 1, 20], [dev(cols[2]), dev(cols[3]), dev(v)])
    t = sess.join(L, R, 0)
    got = sess.to_numpy(t)
    sess.free(t)
    sess._keep.clear()
    k, i, j = rows_of(cols[0] * 40 + cols[1], cols[2] * 40 + cols[3], 2, 1)
    assert np.array_equal(got[0], k // 40) and np.array_equal(got[1], k % 40)
    assert np.array_equal(got[2], v[i]) and np.array_equal(got[3], v[j])
