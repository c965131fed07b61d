"""Decode attention with a workgroup to a (row, kv head) pair, longest rows first: the rank that the embedding kernels write (more rows than
lanes of a wave, equal contexts, every arrangement) and the rule for heads of 128 on either side, against the balanced stream and the
oracle, with the bars of the short-context tests."""
import numpy as np
import pytest

from paper_2506_24119_amd import inputs as si
from test_gpu_decode_short import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [si.WEIGHT_BF16, si.WEIGHT_FP32])
@pytest.mark.parametrize("rows,lens", [
    (33, lambda b: 40), (97, lambda b: 1 + b), (130, lambda b: 130 - b), (260, lambda b: 1 + (37 * b) % 90)])
def test_rows_in_any_order(rows, lens, dtype):
    """264 to 2,080 pairs: below and above the 768 places, one to three rounds of rows; contexts equal, rising, falling and mixed"""
    g = si.ModelGeometry("order", 1, 128, 8, 8, 128, 128, 256, 1e4, weight_dtype=dtype)
    _compare(g, si.make_weights(g, seed=87), [lens(b) for b in range(rows)], True, (0, rows // 2, rows - 1))


@pytest.mark.parametrize("rows,longest,direct", [(40, 600, True), (40, 1100, False), (7, 300, False), (8, 300, True)])
def test_one_long_row(rows, longest, direct):
    """The others wait for it: 320 pairs with one row of 38 pages (estimated 6.8 us) and of 69 (15.3); and from a quarter of the CUs in pairs
    on 19 pages are few (2.7)."""
    g = si.ModelGeometry("order", 1, 128, 16, 8, 128, 128, 256, 1e4, qk_norm=True)
    _compare(g, si.make_weights(g, seed=88), [90 + b % 7 for b in range(rows - 1)] + [longest], direct, (0, rows - 1))
