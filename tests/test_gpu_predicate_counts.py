"""Distinct counts per predicate against numpy, where the predicates of a wave's
2,048 rows or of a block's 32,768 pass from one way of counting to the next."""
import numpy as np
import pytest

from paper_1702_03484_amd import binding as B
from tests.conftest import announce

pytestmark = pytest.mark.gpu

SHAPES = {  # rows of each predicate
    "one": [70_000],
    "wave_border": [2_047, 2, 2_047, 1, 28_671, 1, 40_000],
    "sixteen_a_wave": [128] * 300,
    "seventeen_a_wave": [121] * 300,
    "1024_a_block": [32] * 1_024,
    "1025_a_block": [31] * 1_025,
    "tiny_then_large": [1] * 1_100 + [40_000, 3, 30_000],
    "a_row_each": [1] * 4_096,
}


@pytest.mark.parametrize("values", [1, 7, 5_000])
@pytest.mark.parametrize("shape", SHAPES)
def test_counts_match_numpy(sess, shape, values):
    announce(f"predicate counts {shape} {values}")
    sizes = np.array(SHAPES[shape])
    r = np.random.default_rng(3)
    p = np.repeat(np.arange(sizes.size, dtype=np.int32) + 5_000, sizes)
    p = p[r.permutation(p.size)]
    s, o = (r.integers(0, values, p.size).astype(np.int32) for _ in range(2))
    sess.load(s, p, o)
    got = np.array([B.mapsq_predicate_stats(sess.ctx, 5_000 + q) for q in range(sizes.size)])

    def distinct(x):
        pairs = np.unique(p.astype(np.int64) << 32 | x)
        return np.bincount((pairs >> 32) - 5_000, minlength=sizes.size)

    assert np.array_equal(got, np.stack([sizes, distinct(s), distinct(o)], 1))
