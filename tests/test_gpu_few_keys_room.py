"""The counting shuffle of a few-key LEFT side by its value columns (none to
three LEFT, none to two RIGHT), under allocations that fail, and in arenas that
get tighter: where the sort of the same records has its room the query has,
and its rows are the sort's."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from paper_1702_03484_amd.engine import MapSQ
from tests.conftest import announce

pytestmark = pytest.mark.gpu
IDS = 4_000_000
P1, P2, P3, P4, C = (IDS + 1 + k for k in range(5))
X, Y, Z, W, V, Q = -1, -2, -3, -4, -5, -6
MEMORY = (B.MAPSQ_ERR_CAPACITY, B.MAPSQ_ERR_TOO_LARGE)


def store(left, keys, n3):
    """left = 0: x p1 C (10 rows a key), x p2 C (600 a key): rows of x alone.
    left = 2, 3: x p1 y, w p2 y (and v p4 y).  p3: n3 rows, half of the x's,
    with a z and with C."""
    g = torch.Generator().manual_seed(keys + left)
    x = torch.randperm(IDS, generator=g)[:keys]
    rows = []

    def add(s, p, o):
        rows.append((s, torch.full_like(s, p), o if torch.is_tensor(o) else torch.full_like(s, o)))

    if left == 0:
        add(x.repeat(10), P1, C)
        add(x.repeat((1 << 20) // (16 * keys) + 40), P2, C)
    else:
        add(x, P1, torch.arange(keys) % 8)
        fan = {2: (1 << 20) // keys + 60, 3: 20}[left]
        add(torch.randint(0, IDS, (8 * fan,), generator=g), P2, torch.arange(8).repeat(fan))
        if left == 3:
            fan = (1 << 20) // (20 * keys) + 60
            add(torch.randint(0, IDS, (8 * fan,), generator=g), P4, torch.arange(8).repeat(fan))
    x3 = torch.randint(0, IDS, (n3,), generator=g)
    x3 = x3[~torch.isin(x3, x)]
    have = x[: keys // 2]
    x3 = torch.cat([x3, have, have[: keys // 4]])
    add(x3, P3, torch.randint(0, IDS, x3.shape, generator=g))
    add(x3, P3, C)
    s, p, o = (torch.cat([r[i] for r in rows]) for i in range(3))
    at = torch.randperm(s.numel(), generator=g)
    return [c[at].to(torch.int32).cuda() for c in (s, p, o)]


def patterns(left, right):
    q = {0: [(X, P1, C), (X, P2, C)], 2: [(X, P1, Y), (W, P2, Y)], 3: [(X, P1, Y), (W, P2, Y), (V, P4, Y)]}[left]
    return [*q, {0: (X, P3, C), 1: (X, P3, Z), 2: (X, Q, Z)}[right]]


def rows(sess, q, few):
    """the query's rows, by counting where its rule says so or by the sort alone"""
    sess.set_join_options(semijoin=0 if few else 1, merge=1)  # merge: a LEFT side of x alone is in key order
    try:
        t = sess.query(q)
        got = list(t.vars), [sess.column(t, c).clone() for c in range(t.ncols)]
        sess.free(t)
        return got
    finally:
        sess.set_join_options()


def same(a, b):
    return a[0] == b[0] and all(torch.equal(x, y) for x, y in zip(a[1], b[1]))


@pytest.mark.parametrize("left,right", [(0, 0), (0, 1), (2, 0), (2, 2), (3, 0), (3, 1), (3, 2)])
@pytest.mark.parametrize("keys", [17, 1000])
def test_value_columns(sess, left, right, keys):
    if left == 0:
        keys = min(keys, 100)  # the bound is p1's rows, ten a key
    announce(f"few keys: {keys} keys, {left} + {right} value columns")
    sess.load(*store(left, keys, 700_000))
    q = patterns(left, right)
    got = rows(sess, q, True)
    st = sess.stats()
    assert st.passes == 1 and st.path == B.MAPSQ_PATH_SEMIJOIN and st.left_rows >= 1 << 19
    want = rows(sess, q, False)
    assert sess.stats().path == B.MAPSQ_PATH_SORT and len(want[1][0]) > 0
    assert same(got, want)


def test_one_key_too_many(sess):
    announce("few keys: 1,024 keys take the sort")
    sess.load(*store(2, 1024, 700_000))
    got = rows(sess, patterns(2, 1), True)
    assert sess.stats().passes > 1 and sess.stats().left_rows >= 1 << 19
    assert same(got, rows(sess, patterns(2, 1), False))


def test_failed_allocations():
    announce("few keys: alloc faults")
    q = patterns(2, 2)
    with MapSQ(arena_bytes=1 << 30) as s:
        s.load(*store(2, 300, 700_000))
        want = rows(s, q, False)
        assert same(rows(s, q, True), want) and s.stats().passes == 1  # status words have grown, too
        torch.cuda.synchronize()
        free = B.mapsq_arena_free_bytes(s.ctx)[0]
        failed = by_sort = by_count = 0
        for k in range(40):
            B.mapsq_debug_fail_alloc(s.ctx, k)
            try:
                got = rows(s, q, True)
            except B.MapSQError as e:
                assert e.code in MEMORY, (k, str(e))
                failed += 1
            else:
                assert same(got, want), k
                by_count += s.stats().passes == 1
                by_sort += s.stats().passes > 1
            finally:
                B.mapsq_debug_fail_alloc(s.ctx, -1)
            torch.cuda.synchronize()
            assert B.mapsq_arena_free_bytes(s.ctx)[0] == free, k
        # six scratch blocks and the result, each followed by the sort
        assert failed and by_sort >= 7 and by_count, (failed, by_sort, by_count)


@pytest.mark.parametrize("holes", [False, True])
def test_tighter_arenas(holes):
    """free space in one piece, or with a piece of it apart"""
    announce(f"few keys in tighter arenas, holes={holes}")
    q = patterns(2, 1)
    outcomes = set()
    with MapSQ(arena_bytes=256 << 20) as s:
        s.load(*store(2, 300, 700_000))
        want = rows(s, q, False)
        assert same(rows(s, q, True), want)
        small = torch.zeros(1, dtype=torch.int32, device="cuda")
        for mb in range(20, 200, 12):
            torch.cuda.synchronize()
            try:
                s.dict_create(1, mb << 20)
            except B.MapSQError as e:
                assert e.code == B.MAPSQ_ERR_CAPACITY
                break
            held = []
            if holes:  # three tables of 12 MB, the middle one given back
                n = 1 << 10
                a = s.table([0, 1], [small.expand(n).contiguous(), small.expand(n).contiguous()], key_max=0, sorted_col=1)
                b = s.table([0, 2], [small.expand(n).contiguous(), small.expand(n).contiguous()], key_max=0, sorted_col=1)
                try:
                    held = [s.join(a, b, 0) for _ in range(3)]
                    s.free(held.pop(1))
                except B.MapSQError as e:
                    assert e.code in MEMORY
            out = []
            for few in (True, False):
                try:
                    got = rows(s, q, few)
                    assert same(got, want), (mb, few)
                    out.append(True)
                except B.MapSQError as e:
                    assert e.code in MEMORY, (mb, few, str(e))
                    out.append(False)
            assert out[0] or not out[1], f"refused with {mb} MiB taken, though the sort fits"
            outcomes.add(out[0])
            for t in held:
                s.free(t)
            s._keep.clear()
    assert outcomes == {True, False}
