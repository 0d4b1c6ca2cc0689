"""Attention kernels at the edges of their operand tiles (16 columns, 16-row operands, 32-row steps, 64-row tiles): every
pair of query and key counts around them, forward and backward, on both kernel sets, against the oracle with the
tolerances of the other bf16 cases."""
import itertools

import pytest

from paper_2510_18692_amd import binding as mg
from tests.test_gpu_varlen import run_case

pytestmark = pytest.mark.gpu

EDGES = (1, 4, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 129)


@pytest.mark.parametrize("small_rows", [0, 1 << 30])
def test_every_pair_of_edges(small_rows):
    pairs = list(itertools.product(EDGES, EDGES))
    mg.set_small_group_rows(small_rows)
    try:
        run_case([p[0] for p in pairs], [p[1] for p in pairs], 1, 128, "bf16", seed=small_rows & 1)
    finally:
        mg.set_small_group_rows(-1)
