"""Term hashing, comparing and copying at the sizes where their pieces end:
term lengths around 4, 8 and 16 bytes, runs of empty terms longer than a
staging round, terms longer than a block's byte range, totals around a
multiple of that range, and buffers off every alignment."""
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


def terms_of(name):
    r = np.random.default_rng(len(name))
    text = lambda k: r.integers(0, 256, k, dtype=np.uint8).tobytes()  # noqa: E731
    if name == "lengths":  # every length to 40, each also with another first, middle and last byte
        out = []
        for k in range(41):
            a = text(k)
            out += [a, a]
            out += [a[:p] + bytes([a[p] ^ 1]) + a[p + 1:] for p in sorted({0, k // 2, k - 1}) if 0 <= p < k]
        return out
    if name == "empties":  # 512 terms are staged at a time
        return [b"", b"a"] + [b""] * 2000 + [b"bcd"] + [b""] * 513 + [text(9000)] + [b""] * 511 + [b"e", b""]
    if name == "long":  # 8,192 bytes to a block
        return [text(8191), b"x", text(8192), text(40_000), text(3), text(16_385)]
    if name == "one":
        return [text(1)]
    return [text(int(k)) for k in r.integers(0, 70, 9000)]  # mixed


@pytest.mark.parametrize("skew", [0, 1, 8, 15])
@pytest.mark.parametrize("name", ["lengths", "empties", "long", "one", "mixed"])
def test_round_trip(s, name, skew):
    announce(f"dictionary copies: {name}, buffers {skew} bytes past alignment")
    terms = terms_of(name)
    data, off = D.join_terms(terms)
    exp, known = D.encode(terms)
    buf = torch.zeros(len(data) + 16, dtype=torch.uint8, device="cuda")
    buf[skew: skew + len(data)] = torch.from_numpy(np.frombuffer(data, np.uint8).copy()).cuda()
    s.dict_create(len(terms) + 1, len(data) + 16)
    s.dict_encode(np.frombuffer(b"#" * (skew + 1), np.uint8), np.array([0, skew + 1]))  # the store's end is off alignment too
    got, new = s.dict_encode(buf[skew: skew + len(data)], torch.from_numpy(np.asarray(off, np.int64)).cuda())
    lead = b"#" * (skew + 1)
    exp, known = D.encode([lead] + terms)
    assert np.array_equal(got.cpu().numpy(), exp[1:]) and new == len(known) - 1
    # decode every term of the batch to a buffer off alignment; the bytes around it stay
    total = len(data)
    out = torch.full((total + 64,), 7, dtype=torch.uint8, device="cuda")
    pos = torch.empty(len(terms) + 1, dtype=torch.int64, device="cuda")
    ids = got.contiguous()
    assert B.mapsq_dict_decode(s.ctx, ids.data_ptr(), len(terms), B.MAPSQ_DICT_DEVICE_PTRS, pos.data_ptr(),
                               out.data_ptr() + 16 + skew, total) == total
    out = out.cpu().numpy()
    assert out[16 + skew: 16 + skew + total].tobytes() == data
    assert (out[: 16 + skew] == 7).all() and (out[16 + skew + total:] == 7).all()
    assert np.array_equal(pos.cpu().numpy(), np.asarray(off))
    # and the store itself, identifier by identifier
    text, at = s.dict_decode(np.arange(len(known), dtype=np.int32))
    assert D.split_terms(text, at) == known
