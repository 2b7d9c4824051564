"""Which paths get the source-partitioned layout: not those whose rows are so short that a launch is bound by row ends."""
import pytest

import graphgen
from _util import gpu_prepare_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("draws,built", [(1_600_000, False), (6_000_000, True)])  # 4 and 12 entries a row
def test_short_rows_are_not_partitioned(draws, built):
    full = gpu_prepare_full(graphgen.random_graph("rmat", 1 << 20, seed=5, raw_draws=draws))
    for F in (41, 64):
        full.prepare_width(F)
        assert (full.info().part_rows > 0) == built
