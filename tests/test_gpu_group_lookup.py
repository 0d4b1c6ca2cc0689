"""Tile -> group lookup at the edges of its 64-wide steps: every value row of a group holds the group's number
modulo 251 (exact in bf16), so attention returns it for every query whatever the scores are (a mean of equal
values: exact up to one rounding of the weights' sum, bounded by one bf16 step, 2^-8)."""
import numpy as np
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("G", [1, 63, 64, 65, 256, 257, 4096, 4097, 9000])
def test_every_tile_finds_its_group(G, dtype, D):
    rng = np.random.default_rng(G)
    n = rng.integers(0, 4, G)
    n[rng.integers(0, G, 3)] = 300          # a few groups of several tiles
    if n.sum() == 0:
        n[0] = 1
    cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    ids = np.repeat(np.arange(G), n)
    N = int(cu[-1])
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k = (torch.randn((1, N, D), generator=torch.Generator().manual_seed(G + i)).to(tdt).cuda() for i in range(2))
    val = torch.from_numpy((ids % 251).astype(np.float32)).cuda()
    v = val[None, :, None].expand(1, N, D).to(tdt).contiguous()
    c = torch.from_numpy(cu).cuda()
    o, _ = mg.moga_varlen_attn_fwd(q, k, v, c, c, D ** -0.5)
    got = o.float()[0]
    assert torch.all((got - val[:, None]).abs() <= 2 ** -8 * val[:, None]), G
    if G <= 256:
        o2, lse2 = mg.moga_group_attn_fwd(q, k, v, c, D ** -0.5)
        assert torch.equal(o2, o)
