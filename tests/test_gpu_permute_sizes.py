"""The counting sort at the edges of its single-block kernel (4,096 / 8,192 / 16,384 tokens, 32 groups)
and of the chunked kernels (64-token batches, up to 256 groups), with empty groups: whole numbers, compared exactly with a stable sort."""
import numpy as np
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 5, 32, 33, 256])
@pytest.mark.parametrize("N", [1, 64, 65, 4096, 4097, 8192, 8193, 16384, 16385, 33000])
def test_permutation_is_the_stable_sort(N, M):
    rng = np.random.default_rng(N * 1000 + M)
    group = (rng.random(N) ** 2 * (M if M < 32 else M - 3)).astype(np.int32)   # unbalanced; empty groups for large M
    group[rng.integers(0, N)] = -4                                             # clamped into range
    group[rng.integers(0, N)] = M + 9
    out = mg.moga_permute(torch.from_numpy(group).cuda(), M)
    torch.cuda.synchronize()
    g = np.clip(group, 0, M - 1)
    perm = np.argsort(g, kind="stable")
    inv = np.empty(N, np.int64)
    inv[perm] = np.arange(N)
    counts = np.bincount(g, minlength=M)
    np.testing.assert_array_equal(out["counts"].cpu().numpy(), counts)
    np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))
    assert int(out["max_seqlen"]) == counts.max()
    np.testing.assert_array_equal(out["perm"].cpu().numpy(), perm)
    np.testing.assert_array_equal(out["inv_perm"].cpu().numpy(), inv)
