"""Backward calls whose dQ and dK/dV grids fit HIP's limit (fewer than 2^32 threads) each but not together."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


# H heads, `empty` groups without rows before `sizes`: some 9.4 million blocks of 256 threads for dQ and as many for dK/dV (grids
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
