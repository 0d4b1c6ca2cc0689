"""Weight gradient of up to 65,536 tokens: one block or several per 64 columns, around the lines between them and with last blocks that
are not full.  Against the float64 oracle: 1e-4 of the largest gradient, the bound of the router parity tests (two bf16 limbs of dr
err by 2^-16 each, sums of them by less)."""
import math

import numpy as np
import pytest
import torch

from oracle import moga_oracle as orc
from paper_2510_18692_amd import binding as mg
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,M", [
    (17, 256, 8), (2048, 256, 32), (2049, 256, 20), (2049, 512, 1),   # one block; eight, the last one short
    (2049, 6144, 5), (2049, 9216, 4),                                 # room for two; for one
    (16385, 256, 9),                                                  # 61 of 64 blocks
    (8193, 9216, 3), (65536, 256, 32), (65537, 256, 32),              # the other path from 8,192 tokens a block and 65,536 on
])
def test_router_weight_gradient_of_few_blocks(N, d, M):
    print(f"dW few N={N} d={d} M={M}", flush=True)
    g = torch.Generator().manual_seed(N + d + M)
    x = torch.randn((N, d), generator=g).to(torch.bfloat16)
    w = torch.randn((M, d), generator=g) * (2.0 / math.sqrt(d))
    d_gate = torch.randn(N, generator=g)
    probs = torch.softmax(torch.randn((N, M), generator=g), 1)
    gate, group = probs.max(1)
    dev = [t.cuda() for t in (w, probs, group.to(torch.int32), gate, d_gate)]
    d_w, _ = mg.moga_route_bwd(x.cuda(), *dev)
    if N * d > 10_000_000:   # the oracle's arrays would not be small
        dr = (torch.nn.functional.one_hot(group, M) - probs.double()) * (d_gate.double() * gate.double())[:, None]
        ref = (dr.t() @ x.double()).numpy()
    else:
        ref = orc.route_bwd(P.to64(x), P.to64(w), P.to64(probs), group.numpy(), P.to64(gate), P.to64(d_gate))[0]
    if M == 1:   # the softmax of one logit is constant
        assert float(d_w.abs().max()) == 0.0 and float(np.abs(ref).max()) == 0.0
    else:
        P.assert_close_f32(P.to64(d_w), ref, "dW")


@pytest.mark.parametrize("N,token", [(2049, 2048), (2049, 271), (2049, 272)])   # last of all; last and first of a block
def test_infinite_activation_stays_in_its_column(N, token):
    g = torch.Generator().manual_seed(N)
    x = torch.randn((N, 256), generator=g).to(torch.bfloat16)
    probs = torch.softmax(torch.randn((N, 8), generator=g), 1)
    gate, group = probs.max(1)
    hx = x.clone()
    hx[token, 5] = torch.inf
    dev = [t.cuda() for t in (torch.zeros((8, 256)), probs, group.to(torch.int32), gate, torch.rand(N, generator=g) + 0.5)]
    a, b = (mg.moga_route_bwd(t.cuda(), *dev)[0].cpu() for t in (hx, x))
    assert not torch.isfinite(a[:, 5]).any()
    a[:, 5] = b[:, 5]
    assert torch.equal(a, b)
