"""Store loading against numpy: both index orders, the predicate ranges and the
per-predicate distinct counts, at the edges of the index kernels (rows around
a multiple of four and of the counting block, one and many predicates, packed
words of few, exactly 64 and more than 64 bits, host columns and device
columns on and off a 16-byte boundary)."""
import numpy as np
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu
VX, VY = -1, -2  # variables 0 and 1

CASES = [
    # (rows, entities, predicates, first predicate ID, spread of the predicate IDs)
    (1, 1, 1, 0, 1),                          # one triple of zeros: no bits to sort
    (3, 5, 2, 5, 1),
    (4095, 100, 1, 7, 1),                     # one predicate
    (8193, 1 << 16, 5, 1 << 16, 1),           # 2 * 16 + 3 bits: the high half has three
    (2_049, 40, 3, 40, 1),                    # one row past a wave's share
    (65_537, 900, 3, 900, 1),                 # one row past two counting blocks
    (16_385, 50, 700, 50, 1),                 # many predicates in one counting block
    (40_003, 90, 4097, 90, 1),                # more predicates than have statistics
    (20_011, (1 << 29) - 3, 64, 1 << 29, 1),  # 64 bits: the whole word
    (20_011, (1 << 29) + 9, 64, 1 << 30, 1),  # 66 bits: the permutation sort
    (9_001, 1 << 20, 6, 0, 300_000_000),      # wide predicate IDs: 71 bits
]


def store(case, seed):
    n, e, preds, p0, step = case
    r = np.random.default_rng(seed)
    s, o = (r.integers(0, e, n).astype(np.int32) for _ in range(2))
    s[0] = e - 1
    p = (p0 + step * np.minimum(r.geometric(min(1.0, 4.0 / preds), n) - 1, preds - 1)).astype(np.int32)
    p[: min(n, preds)] = p0 + step * np.arange(min(n, preds))
    return s, p, o


@pytest.mark.parametrize("where", ["host", "device", "device_off"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[1]}x{c[2]}")
def test_indexes_match_numpy(sess, case, where):
    announce(f"load {case} {where}")
    s, p, o = store(case, 11)
    cols = (s, p, o)
    if where != "host":
        pad = 1 if where == "device_off" else 0  # a view one element past the allocation's start
        cols = [torch.from_numpy(np.concatenate([np.zeros(pad, np.int32), x])).cuda()[pad:] for x in cols]
    facts = sess.load(*cols)
    preds = np.unique(p)
    assert (facts.n_triples, facts.n_predicates) == (s.size, preds.size)
    assert facts.max_id == max(s.max(), p.max(), o.max())
    pick = preds if preds.size <= 12 else preds[np.linspace(0, preds.size - 1, 12).astype(int)]
    for q in pick:
        m = p == q
        for key, (a, b) in ((0, (s[m], o[m])), (1, (o[m], s[m]))):
            order = np.lexsort((b, a))
            t = sess.map((VX, int(q), VY), key)
            got = sess.to_numpy(t)
            assert np.array_equal(got[0], a[order]) and np.array_equal(got[1], b[order])
        if preds.size <= 4096:
            want = (int(m.sum()), np.unique(s[m]).size, np.unique(o[m]).size)
            assert B.mapsq_predicate_stats(sess.ctx, int(q)) == want
    if preds.size <= 4096:  # every predicate's counts, not the picked ones alone
        got = [B.mapsq_predicate_stats(sess.ctx, int(q)) for q in preds]
        assert sum(g[0] for g in got) == s.size
        assert sum(g[1] for g in got) == np.unique(p.astype(np.int64) << 31 | s).size
        assert sum(g[2] for g in got) == np.unique(p.astype(np.int64) << 31 | o).size


@pytest.mark.parametrize("bad", [-1, (1 << 31) - 1])
@pytest.mark.parametrize("column", [0, 1, 2])
def test_bad_identifiers_are_refused(sess, column, bad):
    announce(f"load with ID {bad} in column {column}")
    cols = [c.copy() for c in store(CASES[3], 5)]
    cols[column][8192] = bad
    for where in (cols, [torch.from_numpy(c).cuda() for c in cols]):
        with pytest.raises(B.MapSQError) as e:
            sess.load(*where)
        assert e.value.code == B.MAPSQ_ERR_INVALID_ARG
