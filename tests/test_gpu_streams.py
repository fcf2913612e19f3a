"""A session on a stream of its own: what a call documents as complete on
return is complete on every stream, and results read through the session are
the rows, however long the session's stream still works on them."""
import numpy as np
import pytest
import torch

from paper_1702_03484_amd.engine import MapSQ
from tests.conftest import announce

pytestmark = pytest.mark.gpu
N = 20_000_000
PRED = 2_000_000


@pytest.fixture(scope="module")
def side():
    """a store whose scan `?x p ?x` keeps half of its rows, on a side stream"""
    stream = torch.cuda.Stream()
    s = MapSQ(arena_bytes=6 << 30, stream=stream)
    g = torch.Generator().manual_seed(5)
    a = torch.randint(0, PRED, (N,), generator=g, dtype=torch.int32)
    b = torch.where(torch.rand(N, generator=g) < 0.5, a, (a + 1) % PRED)
    s.load(a.numpy(), np.full(N, PRED, dtype=np.int32), b.numpy())
    yield s, stream, a[a == b]
    s.close()


@pytest.mark.parametrize("how", ["map", "query"])
def test_a_scan_is_complete_on_return(side, how):
    announce(f"side stream: {how}")
    s, stream, want = side
    pattern = (-1, -2, -1)  # ?x ?p ?x
    for _ in range(3):
        t = s.map(pattern) if how == "map" else s.query([pattern])
        assert stream.query(), "the session's stream still works"
        got = s.column(t, list(t.vars).index(0)).cpu()  # on torch's stream, not the session's
        assert t.owned and t.nrows == want.numel()
        assert torch.equal(got, want)
        s.free(t)


def test_results_are_read_after_the_sessions_stream(side):
    """a join of 2M + 2M rows: its rows are under way when the call returns"""
    announce("side stream: to_numpy of a join")
    s, stream, _ = side
    k = torch.arange(2_000_000, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    L, R = s.table([0, 1], [k, k * 2], key_max=k.numel()), s.table([0, 2], [k.flip(0), k * 3], key_max=k.numel())
    torch.cuda.synchronize()
    for _ in range(3):
        t = s.join(L, R, 0)
        key, a, b = s.to_numpy(t)
        assert stream.query()
        assert np.array_equal(key, np.arange(k.numel())) and np.array_equal(a, key * 2)
        assert np.array_equal(b, (k.numel() - 1 - key) * 3)
        s.free(t)
    s._keep.clear()
