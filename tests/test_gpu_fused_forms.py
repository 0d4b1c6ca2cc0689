"""The gather-fused backward with dQ and dK/dV in one launch and in one each, with each size of block, against float64."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


# heads, group sizes, (query rows, keys) of the blocks, in one launch.  Apart: ten rounds of blocks and more (short groups of many heads: remainders
# of tiles)
@pytest.mark.parametrize("H,sizes,rows,keys,together", [
    (3, [700, 0, 33, 385], 256, 128, True), (16, [1536, 1300, 1700, 1608], 384, 192, True),
    (4096, [219], 256, 128, False), (4096, [130, 70], 256, 128, False), (4096, [191], 256, 192, False),
    (512, [429, 0, 858], 256, 192, False), (3000, [303], 384, 192, False), (512, [1283], 384, 192, False),
    (12, [5100], 256, 128, True), (5, [3100, 2900, 0, 6384], 256, 128, True), (3, [5400, 5600], 256, 128, True), (6, [5500, 5301], 384, 192, True),
    (12, [5800, 5755], 384, 192, True),
])
def test_fused_backward_in_either_form(H, sizes, rows, keys, together):
    print(f"fused H={H} sizes={sizes}", flush=True)
    N, M, D = sum(sizes), len(sizes), 128
    took = mg.attn_blocks(mg.OP_FUSED_ATTN_BWD, N, N, H, M, 0)
    assert took == ((rows, 2, keys, 2) if together else (rows, 0, keys, 0))
    g = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, d_o = (torch.randn((N, H, D), generator=g, device="cuda").bfloat16() for _ in range(4))
    gate = torch.rand(N, generator=g, device="cuda") + 0.2
    group = torch.repeat_interleave(torch.arange(M, device="cuda"), torch.tensor(sizes, device="cuda"))
    group = group[torch.randperm(N, generator=g, device="cuda")].int()
    pm = mg.moga_permute(group, M)
    o, lse = mg.moga_fused_attn_fwd(q, k, v, pm["perm"], gate, pm["cu_seqlens"], D ** -0.5)
    *got, d_gate = mg.moga_fused_attn_bwd(d_o, q, k, v, o, lse, pm["perm"], pm["inv_perm"], gate, pm["cu_seqlens"], D ** -0.5)
    for h in sorted({0, H // 2, H - 1}):
        want = [torch.zeros((N, D), dtype=torch.double, device="cuda") for _ in range(3)]
        for i in range(M):
            t = (group == i).nonzero()[:, 0]
            q64, k64, v64, g64 = (x[t, h].double() for x in (q, k, v, d_o))
            g64 = g64 * gate[t].double()[:, None]
            p = torch.softmax(D ** -0.5 * (q64 @ k64.T), dim=1)
            ds = p * (g64 @ v64.T - (g64 * (p @ v64)).sum(1, keepdim=True))
            want[0][t], want[1][t], want[2][t] = D ** -0.5 * (ds @ k64), D ** -0.5 * (ds.T @ q64), p.T @ g64
        for x, w in zip(got, want):
            assert (x[:, h].double() - w).norm() <= 1e-2 * w.norm()
            # every row: none of a tile's remainder is left out
            assert bool(((x[:, h].double() - w).norm(dim=1) <= 5e-2 * w.norm(dim=1) + 1e-2 * w.norm() / N ** 0.5).all())
    want = sum((a.double() * b.double()).sum((1, 2)) for a, b in zip(d_o.split(1024, 1), o.split(1024, 1))) / gate.double()
    assert (d_gate.double() - want).norm() <= 1e-4 * want.norm()
