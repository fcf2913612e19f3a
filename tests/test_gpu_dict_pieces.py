"""Term copies by the size of the output: the bytes a block takes grow from 512
to 8,192 as the output grows from half a megabyte to 8.  Totals around the
steps, terms shorter and longer than a piece, buffers off alignment."""
import numpy as np
import pytest
import torch

from oracle import dictionary as D
from paper_1702_03484_amd import binding as B
from paper_1702_03484_amd.engine import MapSQ
from tests.conftest import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def s():
    with MapSQ(arena_bytes=1 << 30) as m:
        yield m


def terms_of(total, longest):
    """terms of 0 to `longest` bytes, `total` in all"""
    r = np.random.default_rng(total)
    cut = np.unique(np.concatenate([[0, total], np.cumsum(r.integers(0, longest + 1, 2 * total // longest + 2))]))
    cut = cut[cut <= total]
    text = r.integers(0, 256, total, dtype=np.uint8).tobytes()
    return [b""] + [text[a:b] for a, b in zip(cut[:-1], cut[1:])] + [b""]


@pytest.mark.parametrize("skew", [0, 5])
@pytest.mark.parametrize("total,longest", [
    (1, 1), (511, 3), (512, 3), (513, 700), (4099, 5), (512 * 1024 - 3, 40), (512 * 1024 + 16 * 1024, 2000),
    (528 * 1024 + 1, 33), ((1 << 20) + 7, 9), ((8 << 20) - 11, 120), ((8 << 20) + 16 * 1024 + 5, 120)])
def test_round_trip(s, total, longest, skew):
    announce(f"dictionary pieces: {total} bytes, terms to {longest}, {skew} bytes past alignment")
    terms = terms_of(total, longest)
    data, off = D.join_terms(terms)
    assert len(data) == total
    exp, known = D.encode([b"#" * (skew + 1)] + terms)
    s.dict_create(len(terms) + 1, total + 16)
    s.dict_encode(np.frombuffer(b"#" * (skew + 1), np.uint8), np.array([0, skew + 1]))
    got, new = s.dict_encode(np.frombuffer(data, np.uint8), np.asarray(off, np.int64))
    assert np.array_equal(got, exp[1:]) and new == len(known) - 1
    out = torch.full((total + 64,), 7, dtype=torch.uint8, device="cuda")
    pos = torch.empty(len(terms) + 1, dtype=torch.int64, device="cuda")
    ids = torch.from_numpy(got.copy()).cuda()
    assert B.mapsq_dict_decode(s.ctx, ids.data_ptr(), len(terms), B.MAPSQ_DICT_DEVICE_PTRS, pos.data_ptr(),
                               out.data_ptr() + 16 + skew, total) == total
    out = out.cpu().numpy()
    assert out[16 + skew: 16 + skew + total].tobytes() == data
    assert (out[: 16 + skew] == 7).all() and (out[16 + skew + total:] == 7).all()
    assert np.array_equal(pos.cpu().numpy(), np.asarray(off))
