"""Router kernels at the edges of their splits, against the float64 oracle.  fp32 sums over N tokens (dW) or d
channels (logits): the bounds are those of the router parity tests (1e-4 of the largest gradient, 2e-5 absolute on
logits of a few units), far above the few 1e-6 that fp32 rounding of such sums shows."""
import math

import numpy as np
import pytest
import torch

from oracle import moga_oracle as orc
from paper_2510_18692_amd import binding as mg
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,M,dtype", [
    (64, 64, 8, "f32"),         # one tile, one column block, eight groups
    (65, 65, 9, "f32"),         # one row, one column, one group more
    (129, 100, 32, "bf16"),     # FMA path with bf16 activations
    (200, 96, 33, "f32"),       # two group blocks, the second with one group
    (20000, 64, 3, "f32"),      # more tiles than splits
    (129, 256, 8, "bf16"),      # matrix-core path: partial sums of 8, 16 and 32 groups per column
    (1000, 512, 9, "bf16"),
    (16385, 256, 17, "bf16"),   # at least 512 tokens a split
])
def test_router_weight_gradient_splits(N, d, M, dtype):
    print(f"dW N={N} d={d} M={M} {dtype}", flush=True)
    g = torch.Generator().manual_seed(N + d + M)
    x = torch.randn((N, d), generator=g).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w = torch.randn((M, d), generator=g) * (2.0 / math.sqrt(d))
    d_gate = torch.randn(N, generator=g)
    rt = orc.route(P.to64(x), P.to64(w))
    dW, _, _ = orc.route_bwd(P.to64(x), P.to64(w), rt["probs"], rt["group"], rt["gate"], P.to64(d_gate))
    dev = [torch.from_numpy(np.ascontiguousarray(rt[k])).cuda() for k in ("probs", "group", "gate")]
    d_w, _ = mg.moga_route_bwd(x.cuda(), w.cuda(), *dev, d_gate.cuda())
    torch.cuda.synchronize()
    P.assert_close_f32(P.to64(d_w), dW, "dW")


@pytest.mark.parametrize("N,d,M,dtype", [(65, 64, 8, "f32"), (200, 96, 33, "f32"), (129, 100, 32, "bf16")])
def test_infinity_in_the_last_token_stays_one(N, d, M, dtype):
    """The last tile of 64 tokens is not full: an infinite activation of the last token makes its column of dW infinite
    with the sign of dr, as the sum says, and no other column changes."""
    g = torch.Generator().manual_seed(N)
    x = torch.randn((N, d), generator=g).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    probs = torch.softmax(torch.randn((N, M), generator=g), 1)
    group = probs.argmax(1).to(torch.int32)
    gate = probs.max(1).values
    d_gate = torch.rand(N, generator=g) + 0.5
    hx = x.clone()
    hx[N - 1, 5] = torch.inf
    dev = [t.cuda() for t in (torch.zeros((M, d)), probs, group, gate, d_gate)]
    a, b = (mg.moga_route_bwd(t.cuda(), *dev)[0].cpu() for t in (hx, x))
    sign = torch.where(torch.arange(M) == group[N - 1], torch.inf, -torch.inf)
    assert torch.equal(a[:, 5], sign)
    a[:, 5] = b[:, 5]
    assert torch.equal(a, b)
