"""Calls at HIP's limit for a grid, fewer than 2^32 threads: of more it launches what is left of the number in 32 bits."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


# Backward calls whose dQ and dK/dV fit each but not together.  H heads, `empty` groups without rows before `sizes`: some 9.4 million blocks of 256 threads for dQ and as many for dK/dV (grids
# are sized by the number of groups); fp32 with the rows that make the difference to blocks of 512 threads
@pytest.mark.parametrize("H,empty,sizes,D,dtype", [(9, 1 << 20, [100, 300, 112], 128, torch.bfloat16),
                                                   (9, 1 << 20, [100, 300, 112], 64, torch.float32),
                                                   (8, (1 << 20) - (1 << 14) - 128, [3072] * 128, 64, torch.float32)])
def test_backward_of_very_many_groups(H, empty, sizes, D, dtype):
    g = torch.Generator(device="cuda").manual_seed(H + D)
    N, scale = sum(sizes), D ** -0.5
    q, k, v, d_o = (torch.randn((H, N, D), generator=g, device="cuda").to(dtype) for _ in range(4))
    few = torch.tensor([0, *sizes], device="cuda").cumsum(0).to(torch.int32)
    many = torch.cat([torch.zeros(empty, dtype=torch.int32, device="cuda"), few])
    try:
        mg.set_small_group_rows(1 << 40)   # for both group counts
        oh, lse = mg.moga_varlen_attn_fwd(q, k, v, few, few, scale)
        want = mg.moga_varlen_attn_bwd(d_o, q, k, v, oh, lse, few, few, scale)   # against the oracle elsewhere
        got = mg.moga_varlen_attn_bwd(d_o, q, k, v, oh, lse, many, many, scale)
    finally:
        mg.set_small_group_rows(-1)
    for x, y in zip(got, want):
        assert torch.equal(x, y)


# A thread per 16 bytes of a row: 2^32 at 64 GiB (one tensor serves as Q, O and dO; one key per group)
def test_row_constants_of_a_64_gib_tensor():
    G, rows, D = 2048, 65536, 128
    N, scale = G * rows + 48, D ** -0.5
    x = torch.empty((1, N, D), device="cuda").uniform_(-1, 1)
    k, v = (torch.randn((1, G, D), device="cuda") for _ in range(2))
    cu_q = torch.tensor([g * rows for g in range(G)] + [N], dtype=torch.int32, device="cuda")
    cu_k = torch.arange(G + 1, dtype=torch.int32, device="cuda")
    d_q = mg.moga_varlen_attn_bwd(x, x, k, v, x, torch.zeros((1, N), device="cuda"), cu_q, cu_k, scale)[0]
    for a, b, g in ((0, 4096, 0), (N // 2, N // 2 + 4096, G // 2), (N - rows, N, G - 1)):
        t = x[0, a:b].double()
        ds = torch.exp(scale * (t @ k[0, g].double())) * (t @ v[0, g].double() - (t * t).sum(1))
        want = scale * ds[:, None] * k[0, g].double()
        assert (d_q[0, a:b] - want).norm() <= 1e-5 * want.norm()   # fp32 sums of 128 products
    del x, d_q
    torch.cuda.empty_cache()


def test_gradients_of_keys_without_queries_above_16_gib():
    H, Nk = 5, (1 << 24) - 1
    q = torch.empty((H, 0, 128), dtype=torch.bfloat16, device="cuda")
    k = torch.empty((H, Nk, 128), dtype=torch.bfloat16, device="cuda")
    old = [torch.ones_like(k) for _ in range(2)]
    del old   # the gradients' memory
    cu_q, cu_k = (torch.tensor([0, n], dtype=torch.int32, device="cuda") for n in (0, Nk))
    d_k, d_v = mg.moga_varlen_attn_bwd(q, q, k, k, q, torch.empty((H, 0), device="cuda"), cu_q, cu_k, 1.0)[1:]
    for t in (d_k, d_v):
        for h in range(H):
            assert not t[h].any()
    del q, k, d_k, d_v
    torch.cuda.empty_cache()


def test_router_with_a_wave_per_token_at_2_to_the_26_tokens():
    N, d, M = (1 << 26) + 5, 4, 2
    x = torch.randn((N, d), device="cuda")
    w = torch.randn((M, d), device="cuda")
    bias = torch.randn(M, device="cuda")
    group, gate, probs, logits = mg.moga_route(x, w, bias, want_logits=True)
    for n in (0, 1 << 25, N - 5000):
        got = mg.moga_route(x[n:n + 5000].clone(), w, bias, want_logits=True)
        for a, b in zip((group, gate, probs, logits), got):
            assert torch.equal(a[n:n + 5000], b)
    assert torch.equal(group, (logits[:, 1] > logits[:, 0]).int())


@pytest.mark.parametrize("D,dtype", [(128, torch.bfloat16), (64, torch.float32)])
def test_more_tiles_than_a_grid_holds_are_refused(D, dtype):
    H, N, G = 2, 300, 1 << 24
    t = torch.randn((H, N, D), device="cuda").to(dtype)
    lse = torch.zeros((H, N), device="cuda")
    cu = torch.zeros(G + 1, dtype=torch.int32, device="cuda")
    cu[-1] = N
    for call in (lambda: mg.moga_varlen_attn_fwd(t, t, t, cu, cu, 0.1), lambda: mg.moga_varlen_attn_bwd(t, t, t, t, t, lse, cu, cu, 0.1)):
        with pytest.raises(mg.MogaError, match="MOGA_ERR_UNSUPPORTED"):
            call()


# Both kernels of the gather-fused backward fit a grid each, and not one together: blocks are counted by groups x heads, most of them empty here.
# By rounds of blocks the call would be launched together (30 tokens) or apart (100)
@pytest.mark.parametrize("N", [30, 100])
def test_gather_fused_backward_of_many_heads_and_groups(N):
    H, M, D = 20000, 256, 128
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, d_o = (torch.randn((N, H, D), generator=g, device="cuda").bfloat16() for _ in range(4))
    group = torch.arange(N, device="cuda").int() % 7 * 30
    gate = torch.rand(N, generator=g, device="cuda") + 0.2
    pm = mg.moga_permute(group, M)
    o, lse = mg.moga_fused_attn_fwd(q, k, v, pm["perm"], gate, pm["cu_seqlens"], D ** -0.5)
    *got, d_gate = mg.moga_fused_attn_bwd(d_o, q, k, v, o, lse, pm["perm"], pm["inv_perm"], gate, pm["cu_seqlens"], D ** -0.5)
    other = (group[:, None] != group[None, :]).cpu()
    for h in (0, 7777, H - 1):
        q64, k64, v64 = (t[:, h].double().cpu().requires_grad_(True) for t in (q, k, v))
        p = torch.softmax((q64 @ k64.T * D ** -0.5).masked_fill(other, float("-inf")), dim=1)
        want = torch.autograd.grad(gate.double().cpu()[:, None] * (p @ v64), (q64, k64, v64), d_o[:, h].double().cpu())
        for x, w in zip(got, want):
            assert (x[:, h].double().cpu() - w).norm() <= 1e-2 * w.norm()
    want = sum((a.double() * b.double()).sum((1, 2)) for a, b in zip(d_o.split(2000, 1), o.split(2000, 1))) / gate.double()
    assert (d_gate.double() - want).norm() <= 1e-4 * want.norm()   # the same products in fp32
