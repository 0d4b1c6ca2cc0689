"""The attention calls that also write their rows in token order give the bits of the calls they stand for."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu

LARGE, SMALL = 0, 1 << 40   # set_small_group_rows: always the one or the other set of bf16 kernels

# N, H, D, groups, dtype: a single row; tiles and groups with remainders, an empty group
SHAPES = [(1, 1, 128, 1, torch.bfloat16), (1, 2, 64, 3, torch.float32), (333, 3, 64, 5, torch.float32), (1000, 2, 128, 4, torch.float32),
          (1560, 4, 128, 8, torch.bfloat16), (2500, 5, 128, 2, torch.bfloat16), (9000, 3, 128, 2, torch.bfloat16),
          (8000, 3, 128, 1, torch.bfloat16), (11201, 3, 128, 3, torch.bfloat16)]
SPLIT_BACKWARD = {(9000, 3, 2), (8000, 3, 1), (11201, 3, 3)}   # N, H, groups: dQ and dK/dV apart with pieces of a last round; the others together


@pytest.fixture
def kernel_set(request):
    mg.set_small_group_rows(request.param)
    yield request.param
    mg.set_small_group_rows(-1)


def splits_a_round(op, N, H, M):
    size = (N, H, 128, M, 0, mg.MOGA_BF16)
    return mg.load().moga_workspace_preferred_bytes(op, N, *size) > mg.workspace_bytes(op, *size)


@pytest.mark.parametrize("kernel_set, N, H, D, M, dtype", [(s, *shape) for shape in SHAPES for s in (LARGE, SMALL) if shape[-1] == torch.bfloat16 or s == SMALL],
                         indirect=["kernel_set"])
def test_token_order_rows_are_those_of_the_separate_calls(kernel_set, N, H, D, M, dtype):
    if dtype == torch.bfloat16:   # the large-group kernels split a round forward at all of these sizes, the others never
        assert splits_a_round(mg.OP_ATTN_FWD, N, H, M) == (kernel_set == LARGE)
        assert splits_a_round(mg.OP_ATTN_BWD_JOINT, N, H, M) == (kernel_set == LARGE and (N, H, M) in SPLIT_BACKWARD)
        ws = mg.load().moga_workspace_preferred_bytes(mg.OP_ATTN_BWD_JOINT, N, N, H, 128, M, 0, mg.MOGA_BF16)
        together = 2 in mg.attn_blocks(mg.OP_ATTN_BWD_JOINT, N, N, H, M, ws)
        assert together == (kernel_set == LARGE and (N, H, M) not in SPLIT_BACKWARD)
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, d_o = (torch.randn((N, H, D), generator=g, device="cuda").to(dtype) for _ in range(4))
    group = torch.randint(0, max(M - 1, 1), (N,), generator=g, device="cuda", dtype=torch.int32)   # the last group stays empty
    gate = torch.rand(N, generator=g, device="cuda") + 0.1
    scale = D ** -0.5
    p = mg.moga_permute(group, M, q, k, v)
    oh, lse = mg.moga_group_attn_fwd(p["qh"], p["kh"], p["vh"], p["cu_seqlens"], scale)
    o = mg.moga_unpermute(oh, p["perm"], gate)
    for got, want in zip(mg.moga_group_attn_fwd_tokens(p["qh"], p["kh"], p["vh"], p["cu_seqlens"], scale, p["perm"], gate), (oh, lse, o)):
        assert torch.equal(got, want)
    d_oh, d_gate = mg.moga_unpermute_bwd(d_o, oh, p["perm"], gate)
    sorted_grads = mg.moga_group_attn_bwd(d_oh, p["qh"], p["kh"], p["vh"], oh, lse, p["cu_seqlens"], scale)
    token_grads = mg.moga_permute_bwd(*sorted_grads, p["perm"])
    for want_sorted in (True, False):
        r = mg.moga_group_attn_bwd_tokens(d_o, p["qh"], p["kh"], p["vh"], oh, lse, p["cu_seqlens"], scale, p["perm"], gate, want_sorted)
        assert torch.equal(r[0], d_oh) and torch.equal(r[1], d_gate)
        for got, want in zip(r[2:5], sorted_grads):
            assert torch.equal(got, want) if want_sorted else got is None
        for got, want in zip(r[5:], token_grads):
            assert torch.equal(got, want)
