"""The blocks that the large bf16 attention kernels take for a call: whole last rounds where the call cannot split them."""
import pytest

from paper_2510_18692_amd import binding as mg


@pytest.fixture
def large_kernels():
    mg.set_small_group_rows(0)
    yield
    mg.set_small_group_rows(-1)


def blocks(op, N, H, M, ws):
    return mg.attn_blocks(op, N, N, H, M, ws)


# N, H, M, query rows where no last round is split: 256 and 384 rows take as many rounds, or 384 fewer
@pytest.mark.parametrize("N,H,M,rows", [
    (5000, 3, 5, 256), (7000, 4, 2, 256), (8348, 12, 8, 256), (40000, 3, 4, 256), (32760, 4, 4, 256), (32760, 4, 8, 256),
    (16384, 4, 2, 256), (8000, 3, 1, 256), (12000, 12, 3, 384), (62400, 12, 5, 384), (99840, 40, 16, 384), (580320, 40, 32, 384),
])
def test_query_rows_of_calls_that_cannot_split(large_kernels, N, H, M, rows):
    for op in (mg.OP_ATTN_FWD, mg.OP_ATTN_BWD):
        need = mg.workspace_bytes(op, N, H, 128, M, 0, mg.MOGA_BF16)
        assert blocks(op, N, H, M, need)[:2] == (rows, False)


@pytest.mark.parametrize("N,H,M,rows", [
    (5000, 3, 5, 128), (7000, 4, 2, 128), (4680, 12, 3, 128), (16384, 4, 2, 128), (8000, 3, 1, 128), (28000, 1, 7, 128),
    (12000, 12, 3, 192), (62400, 12, 5, 192), (99840, 40, 16, 192),
])
def test_key_rows_of_calls_that_cannot_split(large_kernels, N, H, M, rows):
    need = mg.workspace_bytes(mg.OP_ATTN_BWD, N, H, 128, M, 0, mg.MOGA_BF16)
    assert blocks(mg.OP_ATTN_BWD, N, H, M, need)[2:] == (rows, False)


def test_more_groups_than_a_block_looks_up_never_split(large_kernels):
    for op in (mg.OP_VARLEN_ATTN_FWD, mg.OP_VARLEN_ATTN_BWD):
        q, q_split, k, k_split = blocks(op, 300 * 700, 3, 300, 1 << 40)
        assert not q_split and not k_split


# 34 MB past what a call needs hold a round of pieces of 256 rows (or of 128 rows of dV and of dK)
@pytest.mark.parametrize("N,H,M", [(62400, 12, 5), (32760, 12, 8), (12000, 12, 3), (28000, 3, 7), (7000, 4, 2)])
def test_calls_split_with_room_for_short_pieces(large_kernels, N, H, M):
    for op in (mg.OP_ATTN_FWD, mg.OP_ATTN_BWD):
        need = mg.workspace_bytes(op, N, H, 128, M, 0, mg.MOGA_BF16)
        room = 256 + 256 * 256 * 130 * 4
        q, q_split, k, k_split = blocks(op, N, H, M, need + room)
        assert q_split == (q == 256) and k_split == (k == 128)
        assert q_split or blocks(op, N, H, M, need + 2 * room)[0] == 384
        few = mg.load().moga_workspace_preferred_bytes(op, N, N, H, 128, M, 0, mg.MOGA_BF16)
        assert need + room - 512 <= few <= need + room * 3 // 2 + 512
        assert blocks(op, N, H, M, few) == blocks(op, N, H, M, 1 << 40)
    assert blocks(mg.OP_ATTN_FWD, 7000, 4, 2, 256 + 256 * 256 * 130 * 4)[:2] == (256, True)
