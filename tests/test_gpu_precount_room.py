"""The automatic pre-count's sample where it can be wrong: a hot key it does not
look at.  In an arena without room for the sort the exact count runs, so such
a join is refused with its exact size; with room for the sort the count after
it refuses it; nothing else changes its outcome."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from paper_1702_03484_amd.engine import MapSQ
from tests.conftest import announce

pytestmark = pytest.mark.gpu
N = (1 << 23) + 77
RANGE = 1 << 25


def sampled(k):
    """the one key of its block of 64 that the sample counts"""
    return ((k >> 6) * 0x9E3779B1 & 0xFFFFFFFF) >> 26 == k & 63


HOT = next(k for k in range(4711, 5000) if not sampled(k))


def sides(hot):
    g = torch.Generator(device="cuda").manual_seed(3)
    out = []
    for _ in range(2):
        a = torch.randint(0, RANGE, (N,), generator=g, device="cuda", dtype=torch.int32)
        a[:: N // hot] = HOT
        out.append(a)
    return out


def rows_of(a, b):
    return int((torch.bincount(a, minlength=RANGE) * torch.bincount(b, minlength=RANGE)).sum())


# the sort takes 24 bytes of each of 16.8M records (403 MB) and its output,
# with the hot key on 6,000 rows of each side, 38M rows of 12 bytes (457 MB)
@pytest.mark.parametrize("mib,hot,code", [
    (320, 6000, B.MAPSQ_ERR_TOO_LARGE),  # no room for the sort: counted exactly
    (320, 5, B.MAPSQ_ERR_CAPACITY),      # the output would fit, the sort does not
    (800, 6000, B.MAPSQ_ERR_TOO_LARGE),  # sampled, sorted, counted
    (800, 5, B.MAPSQ_OK)])
def test_outcome(mib, hot, code):
    announce(f"pre-count in {mib} MiB, hot key on {hot} rows a side")
    a, b = sides(hot)
    want = rows_of(a, b)
    va = torch.arange(N, dtype=torch.int32, device="cuda")
    with MapSQ(arena_bytes=mib << 20) as s:
        L, R = s.table([0, 1], [a, va], key_max=RANGE - 1), s.table([0, 2], [b, va], key_max=RANGE - 1)
        free = B.mapsq_arena_free_bytes(s.ctx)[0]
        if code == B.MAPSQ_OK:
            t = s.join(L, R, 0)
            assert t.nrows == want == s.stats().out_rows
            k, x, y = (s.column(t, c) for c in range(3))
            assert torch.equal(a[x.long()], k) and torch.equal(b[y.long()], k)
            s.free(t)
        else:
            with pytest.raises(B.MapSQError) as e:
                s.join(L, R, 0)
            assert e.value.code == code and s.stats().out_rows == want
        torch.cuda.synchronize()
        assert abs(B.mapsq_arena_free_bytes(s.ctx)[0] - free) <= 64 << 20  # status words may have grown
