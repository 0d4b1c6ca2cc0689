"""Sort and gather in one launch (up to 16,384 tokens and 32 groups, by the bytes of a token's rows) or two: every integer and
every row against a stable sort."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 15, 16, 17, 255, 257, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 8192, 8193, 16383, 16384, 16385])
@pytest.mark.parametrize("M,H,D,dtype", [(1, 1, 64, torch.float32), (8, 5, 128, torch.bfloat16), (9, 2, 128, torch.float32), (32, 3, 128, torch.bfloat16), (20, 9, 128, torch.bfloat16),
                                         (32, 12, 128, torch.bfloat16), (9, 6, 128, torch.float32),
                                         (8, 16, 128, torch.bfloat16), (20, 12, 128, torch.float32)])   # a block per tensor
def test_sort_and_gather(N, M, H, D, dtype):
    g = torch.Generator(device="cuda").manual_seed(N + M)
    group = torch.randint(-1, M + 1, (N,), generator=g, device="cuda", dtype=torch.int32)   # ids outside are clamped
    q, k, v = (torch.randn((N, H, D), generator=g, device="cuda").to(dtype) for _ in range(3))
    p = mg.moga_permute(group, M, q, k, v)
    ids = group.clamp(0, M - 1).cpu()
    perm = torch.sort(ids, stable=True).indices
    counts = torch.bincount(ids, minlength=M)
    assert torch.equal(p["perm"].cpu().long(), perm)
    assert torch.equal(p["inv_perm"].cpu().long(), torch.argsort(perm))
    assert torch.equal(p["counts"].cpu().long(), counts)
    assert torch.equal(p["cu_seqlens"].cpu().long(), torch.cat([torch.zeros(1, dtype=torch.long), counts.cumsum(0)]))
    assert p["max_seqlen"].item() == counts.max().item()
    for got, src in ((p["qh"], q), (p["kh"], k), (p["vh"], v)):
        assert torch.equal(got.cpu(), src.cpu()[perm].transpose(0, 1))
