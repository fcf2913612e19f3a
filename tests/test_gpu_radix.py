"""The shuffle's radix passes at their edges: remainders of the 16,384- and
32,768-record tiles (32 keys per thread from 25,165,824 records on), the side
boundary inside a tile, histograms of whole and odd tiles on and off a 16-byte
boundary, keys of 1 to 31 bits, carried values and record ids, digit widths of 4
to 11 bits.  Both sides hold every key once, so the rows are known exactly."""
import pytest
import torch

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu
BIG = 3 << 23


def one_to_one(sess, n, top, values, off, tuning=(0, 0)):
    g = torch.Generator(device="cuda").manual_seed(n)
    ids = torch.arange(n, device="cuda", dtype=torch.int64)
    keys = (ids if top < 2 * n else ids * (top // n)).to(torch.int32)
    keys[-1] = top - 1
    sides = []
    for _ in range(2):
        perm = torch.randperm(n, generator=g, device="cuda")
        pad = torch.zeros(off, dtype=torch.int32, device="cuda")
        cols = [torch.cat([pad, keys[perm]])[off:]] + [torch.cat([pad, (perm * 3 + c).to(torch.int32)])[off:]
                                                       for c in range(values)]
        sides.append(cols)
    try:
        sess.set_tuning(*tuning)
        sess.set_join_options(semijoin=1, merge=1, precount=1)
        t = sess.join(sess.table(list(range(1 + values)), sides[0], key_max=top - 1),
                      sess.table([0, *range(20, 20 + values)], sides[1], key_max=top - 1), 0)
        assert sess.stats().path == B.MAPSQ_PATH_SORT and t.nrows == n
        assert torch.equal(sess.column(t, 0), keys)
        for c in range(values):
            want = (ids * 3 + c).to(torch.int32)
            assert torch.equal(sess.column(t, 1 + c), want) and torch.equal(sess.column(t, 1 + values + c), want)
        sess.free(t)
    finally:
        sess.set_tuning()
        sess.set_join_options()
        sess._keep.clear()


@pytest.mark.parametrize("values", [0, 1, 2])
@pytest.mark.parametrize("n,bits,off", [
    (2049, 12, 0), (8191, 13, 1), (8192, 24, 0), (8193, 31, 3), (262_143, 18, 0), (262_145, 30, 1),
    (1_000_003, 20, 0), ((1 << 21) - 1, 22, 2), ((1 << 21) + 1, 31, 0)])
def test_rows(sess, n, bits, off, values):
    announce(f"radix n={n} bits={bits} off={off} values={values}")
    one_to_one(sess, n, 1 << bits if bits < 31 else (1 << 31) - 1, values, off)


@pytest.mark.parametrize("n", [BIG // 2 - 1, BIG // 2, BIG // 2 + 8195])
def test_large_tiles(sess, n):
    announce(f"radix large tiles n={n}")
    one_to_one(sess, n, 1 << 24, 1, n % 3)


@pytest.mark.parametrize("rb", range(4, 12))
@pytest.mark.parametrize("kpt", [8, 16])
def test_digit_widths(sess, rb, kpt):
    announce(f"radix width {rb} kpt {kpt}")
    one_to_one(sess, 40_001, 1 << 27, 1, 1, (rb, kpt))
    one_to_one(sess, 3_000, 1 << 16, 2, 0, (rb, kpt))
