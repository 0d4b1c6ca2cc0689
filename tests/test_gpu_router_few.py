"""Few-token router kernel with four and with eight waves per block (eight: at most 192 blocks of 32 tokens and 2,560 channels or
more) around those lines, against float64: 2e-5 absolute on logits of a few units, the bound of the router parity tests."""
import math

import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 33, 6144, 6145])
@pytest.mark.parametrize("d,M", [(2560, 32), (2560 - 64, 17), (2560 + 64, 1), (5120, 20)])
def test_few_token_router_lines(N, d, M):
    print(f"router N={N} d={d} M={M}", flush=True)
    g = torch.Generator().manual_seed(N + d + M)
    x = torch.randn((N, d), generator=g).to(torch.bfloat16)
    w = torch.randn((M, d), generator=g) * (2.0 / math.sqrt(d))
    b = torch.randn(M, generator=g)
    group, gate, probs, logits = mg.moga_route(x.cuda(), w.cuda(), b.cuda(), want_logits=True)
    ref = x.double() @ w.double().t() + b.double()
    assert float((logits.cpu().double() - ref).abs().max()) <= 2e-5
    torch.testing.assert_close(probs.cpu().double(), torch.softmax(ref, 1), rtol=0, atol=2e-5)
    top, where = ref.max(1)
    clear = torch.ones(N, dtype=torch.bool) if M == 1 else top - ref.topk(2, 1).values[:, 1] > 1e-4
    assert torch.equal(group.cpu().long()[clear], where[clear])
    torch.testing.assert_close(gate.cpu(), probs.cpu().max(1).values, rtol=1e-6, atol=0)
