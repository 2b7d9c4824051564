"""Products over few rows, whose columns are dealt to several workgroups: row counts on both sides of those where a workgroup takes more
of them, widths whose last piece is not full."""
import numpy as np
import pytest

from test_gpu_combination_shapes import _products

pytestmark = pytest.mark.gpu

# rows: one workgroup, then the last and first with 4 and 2, 2 and 1 pieces of four blocks, and with 2 and 1 of two, by either rule
ROWS = (1, 100, 4_096, 4_097, 8_192, 8_193, 12_288, 12_289, 16_384, 16_385)


@pytest.mark.parametrize("Fi,Fo", [(128, 128), (127, 33), (97, 65), (66, 128), (128, 16), (65, 7), (64, 64), (33, 47), (40, 9), (63, 100)])
def test_row_counts_around_the_rules(Fi, Fo):
    order = np.random.default_rng(81).permutation(17_000)
    for m in ROWS:
        _products(17_000, np.sort(order[:m]), Fi, Fo, m)


@pytest.mark.parametrize("m", [24_576, 24_577, 49_152, 49_153])
@pytest.mark.parametrize("Fi,Fo", [(128, 16), (100, 5), (64, 16), (34, 3)])
def test_narrow_rows_onto_wide_ones(Fi, Fo, m):
    _products(50_000, np.sort(np.random.default_rng(82).permutation(50_000)[:m]), Fi, Fo, m)
