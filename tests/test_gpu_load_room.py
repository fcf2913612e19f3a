"""Loading into an arena that has just the room a load needs: the indexes are
those of a load with room to spare."""
import numpy as np
import pytest
import torch

from paper_1702_03484_amd import binding as B
from paper_1702_03484_amd.engine import MapSQ
from tests.conftest import announce

pytestmark = pytest.mark.gpu
IDS = 2_000_000
PREDS = 7


def triples(n):
    rng = np.random.default_rng(n)
    return (rng.integers(0, IDS, n, dtype=np.int32), rng.integers(IDS, IDS + PREDS, n, dtype=np.int32),
            rng.integers(0, IDS, n, dtype=np.int32))


def indexes(sess):
    """both orders of every predicate, and its statistics"""
    out = []
    for p in range(IDS, IDS + PREDS):
        for key in (0, 1):
            t = sess.map((-1, p, -2), key)
            out.append([sess.column(t, c).clone().cpu() for c in range(t.ncols)])
        out.append([torch.tensor(B.mapsq_predicate_stats(sess.ctx, p))])
    return out


def same(a, b):
    return len(a) == len(b) and all(torch.equal(x, y) for p, q in zip(a, b) for x, y in zip(p, q))


@pytest.fixture(scope="module")
def want(sess):
    made = {}

    def of(n):
        if n not in made:
            sess.load(*triples(n))
            made[n] = indexes(sess)
        return made[n]
    return of


# 44 bytes a triple for the columns, the indexes and the sort, and 12 for the
# predicate table, in 64 MiB: 1.17M triples leave 1.0 MB
@pytest.mark.parametrize("n", [1_000_000, 1_170_000])
def test_smallest_arena(want, n):
    announce(f"load of {n} triples into 64 MiB")
    ref = want(n)
    with MapSQ(arena_bytes=64 << 20) as s:
        s.load(*triples(n))
        assert same(indexes(s), ref)


def test_every_failed_allocation(want):
    """an allocation that fails ends in a memory status or in the same indexes"""
    announce("load: alloc faults")
    n = 50_000
    ref = want(n)
    done = failed = 0
    with MapSQ(arena_bytes=256 << 20) as s:
        for k in range(30):
            B.mapsq_debug_fail_alloc(s.ctx, k)
            try:
                s.load(*triples(n))
            except B.MapSQError as e:
                assert e.code == B.MAPSQ_ERR_CAPACITY, (k, str(e))
                failed += 1
                continue
            finally:
                B.mapsq_debug_fail_alloc(s.ctx, -1)
            assert same(indexes(s), ref), k
            done += 1
    assert failed >= 11 and done >= 10
