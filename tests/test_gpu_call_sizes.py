"""Kernels that calls of few rows take, at the edges of their ranges: each against the oracle, or bit for bit against the calls
that it stands for."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg
from tests import test_gpu_backward as tb
from tests import test_gpu_balance as tl
from tests import test_gpu_forward as tf

pytestmark = pytest.mark.gpu


# one row; tiles of 16 rows and steps of 128 (four waves of 32, D = 64) or 64 (D = 128) with remainders; an empty group
@pytest.mark.parametrize("sizes,H,D", [([1], 1, 64), ([15, 16, 17, 0, 31, 32, 33], 2, 64), ([63, 64, 65, 127, 128, 129, 160], 1, 64),
                                       ([15, 16, 17, 0, 31, 32, 33], 2, 128), ([63, 64, 65, 80], 3, 128), ([700, 5], 2, 64)])
def test_fp32_attention(sizes, H, D):
    tf.test_group_attention_forward_matches_oracle(sizes, H, D, "f32")
    tb.test_group_attention_backward_matches_oracle(sizes, H, D, "f32")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n", [5, 37, 64])
def test_fp32_infinite_last_row_is_counted_once(n, D):
    """A group's last row stands in for those past its end, with weight 0: an infinity in it stays one, and no NaN."""
    g = torch.Generator(device="cuda").manual_seed(D + n)
    q, k, v, d = (torch.randn((1, n, D), generator=g, device="cuda") for _ in range(4))
    d[0, n - 1, 3] = float("inf")
    cu = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    dv = mg.moga_group_attn_bwd(d, q, k, v, *mg.moga_group_attn_fwd(q, k, v, cu, D ** -0.5), cu, D ** -0.5)[2]
    assert torch.isinf(dv[0, :, 3]).all() and torch.isfinite(dv[0, :, :3]).all() and torch.isfinite(dv[0, :, 4:]).all()


# blocks of 32 tokens whose four waves share 64-channel blocks: remainders of both, fewer channel blocks than waves, both sides of
# the lines to the other kernel
@pytest.mark.parametrize("N,d,M", [(1, 64, 1), (31, 128, 32), (32, 256, 5), (33, 320, 20), (500, 576, 31), (16384, 192, 8),
                                   (28672, 128, 20), (28673, 128, 20), (32768, 128, 20), (32769, 128, 20), (24576, 128, 20), (24577, 128, 20),
                                   (32896, 256, 20), (32897, 256, 20), (49152, 256, 20), (49153, 256, 20)])
def test_router_of_few_tokens(N, d, M):
    tf.test_route_matches_oracle(N, d, M, "bf16", N % 2 == 1)


# one launch up to 2,048 tokens: sixteen waves of 16 tokens, blocks of 64 columns
@pytest.mark.parametrize("N,d,M", [(1, 256, 1), (15, 256, 32), (17, 512, 5), (255, 256, 9), (257, 256, 31), (2048, 256, 20), (2049, 256, 20)])
def test_router_weight_gradient_of_few_tokens(N, d, M):
    tb.test_route_bwd_matches_oracle(N, d, M, "bf16", False)


# every kernel of the router's backward: the two matrix-core paths, fp32, more than 32 groups, with and without d_x
@pytest.mark.parametrize("N,d,M,dtype,want_dx", [(300, 256, 8, torch.bfloat16, True), (2500, 256, 8, torch.bfloat16, False),
                                                 (300, 100, 40, torch.bfloat16, True), (300, 128, 5, torch.float32, True)])
def test_router_backward_with_the_balancing_term_has_the_bits_of_the_two_calls(N, d, M, dtype, want_dx):
    g = torch.Generator(device="cuda").manual_seed(N + M)
    x = torch.randn((N, d), generator=g, device="cuda").to(dtype)
    w = torch.randn((M, d), generator=g, device="cuda")
    group, gate, probs = mg.moga_route(x, w, want_probs=True)[:3]
    d_gate, d_loss = torch.randn(N, generator=g, device="cuda"), torch.tensor(-1.7, device="cuda")
    _, frac, _ = mg.moga_balance_loss(group, gate, M, 0.1)
    got = mg.moga_route_bwd_balanced(x, w, probs, group, gate, d_gate, frac, 0.1, d_loss, want_dx)
    mg.moga_balance_loss_bwd(group, frac, 0.1, d_loss=d_loss, d_gate=d_gate)
    want = mg.moga_route_bwd(x, w, probs, group, gate, d_gate, want_dx)
    assert torch.equal(got[0], want[0]) and (torch.equal(got[1], want[1]) if want_dx else got[1] is None)


@pytest.mark.parametrize("N,M", [(1, 1), (1023, 256), (8192, 20), (8193, 20)])
def test_balancing_loss_in_one_block(N, M):
    tl.test_balance_loss_matches_oracle(N, M, True)


# bf16: the small-group kernels (`large` False), and the large-group ones with a split round
@pytest.mark.parametrize("N,H,D,dtype,large", [
    (1, 1, 64, torch.float32, False), (17, 5, 128, torch.float32, False), (700, 3, 128, torch.bfloat16, False),
    (2500, 2, 128, torch.bfloat16, False), (700, 3, 128, torch.bfloat16, True), (2500, 2, 128, torch.bfloat16, True)])
def test_branch_rows_and_constants_are_those_of_the_separate_calls(N, H, D, dtype, large):
    try:
        mg.set_small_group_rows(0 if large else 1 << 40)
        branch_rows_and_constants(N, H, D, dtype, large)
    finally:
        mg.set_small_group_rows(-1)


def branch_rows_and_constants(N, H, D, dtype, split):
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, d_o = (torch.randn((N, H, D), generator=g, device="cuda").to(dtype) for _ in range(4))
    inv_m, q_slot = (torch.randperm(N, generator=g, device="cuda").to(torch.int32) for _ in range(2))
    index = torch.randint(0, N, (N + N // 3,), generator=g, device="cuda", dtype=torch.int32)   # keys: some tokens twice, some not at all
    inv_slots = torch.sort(index, stable=True).indices.to(torch.int32)
    inv_cu = torch.cat([torch.zeros(1, device="cuda"), torch.bincount(index, minlength=N).cumsum(0)]).to(torch.int32)
    order = lambda inv: torch.argsort(inv.long()).to(torch.int32)
    rows = lambda src, idx: mg.moga_gather_rows(src, idx)
    ident = torch.arange(N, dtype=torch.int32, device="cuda")
    want = [rows(t, order(inv_m)) for t in (q, k, v)] + [rows(q, order(q_slot)), rows(k, index), rows(v, index)] + [rows(t, ident) for t in (q, k, v)]
    got = mg.moga_gather3_fwd(q, k, v, inv_m, q_slot, inv_cu, inv_slots)
    for a, b in zip(got, want):
        assert torch.equal(a, b)

    cut = lambda n, *parts: torch.tensor([0, *(n * p // 8 for p in parts), n], dtype=torch.int32, device="cuda")
    scale = D ** -0.5
    branches = [(got[0:3], cut(N, 3), cut(N, 3)), (got[3:6], cut(N, 2, 2), cut(index.numel(), 1, 5)), (got[6:9], cut(N, 4, 7), cut(N, 4, 7))]
    gate = torch.rand(N, generator=g, device="cuda") + 0.1
    fwd = [mg.moga_varlen_attn_fwd(*t, cq, ck, scale) for t, cq, ck in branches]
    a = [o for o, _ in fwd]
    want_d = mg.moga_merge3_bwd(d_o, a[0], inv_m, q_slot, None, gate)
    r = mg.moga_merge3_bwd_rows(d_o, *a, inv_m, q_slot, None, gate, [l for _, l in fwd], scale, branches[0][1], branches[1][1], index.numel(),
                                branches[2][1])
    for x, y in zip(r[:4], want_d):
        assert torch.equal(x, y)
    for (t, cq, ck), (o, lse), d, ws in zip(branches, fwd, want_d, r[4:]):
        need = mg.workspace_bytes(mg.OP_VARLEN_ATTN_BWD, N, H, D, cq.numel() - 1, 0, mg.MOGA_BF16 if dtype == torch.bfloat16 else mg.MOGA_F32)
        assert (ws.numel() > need + (32 << 20)) == split   # room for the pieces
        want_g = mg.moga_varlen_attn_bwd(d, *t, o, lse, cq, ck, scale)
        for x, y in zip(mg.moga_varlen_attn_bwd_rows(d, *t, o, lse, cq, ck, scale, ws), want_g):
            assert torch.equal(x, y)
        assert int(mg.attn_bwd_status(ws, N, H)) == 0   # cleared by the merge
