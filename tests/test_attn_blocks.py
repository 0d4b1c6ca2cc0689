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
    (16384, 4, 2, 256), (8000, 3, 1, 256), (12000, 12, 3, 256), (62400, 12, 5, 384), (99840, 40, 16, 384), (580320, 40, 32, 384),
    (48985, 3, 8, 256), (54990, 4, 16, 256),      # 2.2 and 3.4 rounds: 384 rows not by far cheaper
    (12750, 40, 15, 384), (13000, 40, 13, 384),   # more whole rounds than with 256 rows by price, out of step by then
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


# mean rows on either side of the line between the kernels for small groups and the large ones, with and without room to split a round
@pytest.mark.parametrize("H,M,below,above,room", [
    (1, 4, 2700, 2900, True), (1, 2, 4000, None, False), (2, 4, 2000, None, False),        # a third of a round or less
    (4, 20, 1000, 1310, True), (12, 6, 1250, 1310, True), (4, 20, 1250, 1310, False),       # 1.1 to 1.6 rounds
    (40, 33, 440, 460, True), (40, 33, 440, 460, False), (40, 60, 390, 410, True),         # 8.9 and 14
])
def test_backward_line_between_the_kernel_sets(H, M, below, above, room):
    for n, small in ((below, True), (above, False)):
        if n:
            need = mg.workspace_bytes(mg.OP_ATTN_BWD, n * M, H, 128, M, 0, mg.MOGA_BF16)
            took = blocks(mg.OP_ATTN_BWD, n * M, H, M, need + (room << 27))
            assert (took == (128, False, 64, False)) == small, n


def test_calls_take_the_same_kernels_with_the_bytes_they_ask_for():
    """The preferred bytes give the blocks that any amount of room gives, on either side of every line."""
    for op in (mg.OP_ATTN_FWD, mg.OP_ATTN_BWD):
        for H in (1, 4, 12, 40):
            for M in (1, 2, 5, 8, 20, 60):
                for n in range(100, 8400, 150):
                    size = mg.load().moga_workspace_preferred_bytes(op, n * M, n * M, H, 128, M, 0, mg.MOGA_BF16)
                    assert blocks(op, n * M, H, M, size) == blocks(op, n * M, H, M, 1 << 40), (op, H, M, n)


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


def preferred(op, N, H, M):
    return mg.load().moga_workspace_preferred_bytes(op, N, N, H, 128, M, 0, mg.MOGA_BF16)


SMALL, SHORT, LONG = (128, 0, 64, 0), (256, 2, 128, 2), (384, 2, 192, 2)


# dQ and dK/dV of one call: together in one launch of the large kernels, as small blocks, or apart (None: the blocks of the other entry points)
@pytest.mark.parametrize("N,H,M,took", [
    (6900, 3, 3, SMALL), (6800, 3, 4, SMALL), (20791, 1, 11, SMALL),   # 243 to 253 large blocks: a full round, which routed groups exceed
    (13228, 1, 10, SMALL), (14781, 2, 2, None), (5675, 1, 2, None),    # more than five groups, a quarter of a round; long groups
    (8000, 3, 1, None), (24325, 4, 5, None),                           # long groups, whose last rounds are split
    (54400, 3, 16, None), (54384, 3, 16, LONG), (64000, 5, 8, None), (63992, 5, 8, LONG),   # on either side of the line: 2.5 and 4.9 rounds
    (62400, 12, 16, None), (40000, 4, 100, SMALL),                     # ten rounds; the smallest groups
    (4095, 4, 4, SHORT), (9000, 12, 5, LONG), (45453, 4, 16, LONG), (20000, 12, 10, LONG), (15000, 40, 16, LONG),
])
def test_joint_backward_is_launched_in_its_faster_form(N, H, M, took):
    apart = blocks(mg.OP_ATTN_BWD, N, H, M, preferred(mg.OP_ATTN_BWD, N, H, M))
    assert blocks(mg.OP_ATTN_BWD_JOINT, N, H, M, preferred(mg.OP_ATTN_BWD_JOINT, N, H, M)) == (took or apart)


def test_joint_backward_takes_the_same_form_with_the_bytes_it_asks_for():
    for H in (1, 4, 12, 40):
        for M in (1, 2, 5, 8, 20, 60):
            for n in range(100, 8400, 150):
                size = preferred(mg.OP_ATTN_BWD_JOINT, n * M, H, M)
                need = mg.workspace_bytes(mg.OP_ATTN_BWD_JOINT, n * M, H, 128, M, 0, mg.MOGA_BF16)
                took = blocks(mg.OP_ATTN_BWD_JOINT, n * M, H, M, 1 << 40)
                if size > need:   # asked for only if a round is split
                    assert blocks(mg.OP_ATTN_BWD_JOINT, n * M, H, M, size) == took and 1 in (took[1], took[3]), (H, M, n)
                else:
                    assert 1 not in (took[1], took[3]), (H, M, n)


# (queries, groups) of a block's branches: routed groups, windows, frames.  From one to eight rounds of blocks: forward the small kernels for all if a
# branch has short groups, backward for windows of a few tokens; from eight on for windows of less than 300
@pytest.mark.parametrize("T,H,M,window,fwd,bwd", [
    (3, 12, 5, 4, (True, True, True), (False, True, False)), (3, 12, 5, 16, (True, True, True), (False, True, False)),
    (3, 12, 5, 30, (True, True, True), (False, False, False)), (6, 12, 10, 195, (True, True, True), (False, False, False)),
    (6, 12, 10, 780, (True, True, True), (False, False, False)),
    (10, 12, 5, 4, (False, True, False), (False, True, False)), (10, 12, 5, 390, (False, False, False), (False, False, False)),
])
def test_branches_with_small_windows_take_the_small_kernels(T, H, M, window, fwd, bwd):
    N = 1560 * T
    sizes = [(N, M), (N, N // window), (N, T)]
    assert mg.small_calls(mg.OP_VARLEN_ATTN_FWD, sizes, H) == fwd
    assert mg.small_calls(mg.OP_VARLEN_ATTN_BWD, sizes, H) == bwd


def test_long_groups_of_all_branches_take_the_large_kernels():
    sizes = [(37440, 5), (37440, 12), (37440, 24)]   # 7,488, 3,120 and 1,560 rows
    for op in (mg.OP_VARLEN_ATTN_FWD, mg.OP_VARLEN_ATTN_BWD):
        assert mg.small_calls(op, sizes, 3) == (False, False, False)


def test_forward_call_of_long_groups_asks_for_room_to_run_by_itself():
    for N, H, G, alone in ((8300, 3, 1, True), (24960, 4, 2, True), (24960, 4, 8, False), (99840, 12, 1, False)):
        size = (N, H, 128, G, 0, mg.MOGA_BF16)
        assert (mg.load().moga_workspace_preferred_bytes(mg.OP_ATTN_FWD_CALL, N, *size) > mg.workspace_bytes(mg.OP_ATTN_FWD_CALL, *size)) == alone
