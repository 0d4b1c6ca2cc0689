"""The large bf16 kernels at the edges of their tiles: last tiles of a group that take three columns of 16 rows per wave, two, or
leave waves idle, with either number of query rows per block, against the oracle with the tolerances of the other bf16 cases."""
import pytest

from paper_2510_18692_amd import binding as mg
from tests import test_gpu_backward as tb
from tests import test_gpu_forward as tf

pytestmark = pytest.mark.gpu

SIZES = [1, 47, 48, 49, 95, 97, 127, 128, 129, 255, 256, 257, 383, 384, 385, 639, 640, 641, 767, 769]


# one head: 256 query rows per block; two: 384
@pytest.mark.parametrize("H", [1, 2])
def test_forward_at_tile_edges(H):
    mg.set_small_group_rows(0)
    try:
        tf.test_group_attention_forward_matches_oracle(SIZES, H, 128, "bf16")
    finally:
        mg.set_small_group_rows(-1)


# with the key tiles' edges: 256 query rows per block (dQ); without: 384
@pytest.mark.parametrize("more", [[], [31, 33, 63, 65, 96, 143, 144, 145, 191, 192, 193, 320, 321]], ids=["384 rows", "256 rows"])
def test_backward_at_tile_edges(more):
    mg.set_small_group_rows(0)
    try:
        tb.test_group_attention_backward_matches_oracle(SIZES + more, 2, 128, "bf16")
    finally:
        mg.set_small_group_rows(-1)
