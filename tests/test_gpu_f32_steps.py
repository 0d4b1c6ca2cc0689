"""fp32 attention at the lines between one and two 16-row tiles per step (head_dim 64: a mean of 768 streamed rows forward, 2,048
backward) and around the edges of both steps, against the float64 oracle: 1e-4 of the largest value, the bound of the fp32
configuration (fp32 sums of at most 2,100 terms of a convex combination err by a few 1e-6)."""
import numpy as np
import pytest
import torch

from oracle import stga_oracle as sto
from paper_2510_18692_amd import binding as mg
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,nk", [
    ([15, 16, 17, 63, 64, 65], [15, 16, 17, 63, 64, 65]),   # one tile and one round of the four waves
    ([20], [767]), ([20], [768]), ([33, 0], [1, 1536]),     # forward
    ([2048], [40]), ([2049], [40]),                         # backward by its queries
    ([40], [2048]), ([40], [2065]),                         # and by its keys
])
def test_f32_attention_around_the_step_lines(nq, nk):
    print(f"f32 steps nq={nq} nk={nk}", flush=True)
    H, D = 1, 64
    g = torch.Generator().manual_seed(sum(nq) + sum(nk))
    q, dA = (torch.randn((sum(nq), H, D), generator=g) for _ in range(2))
    k, v = (torch.randn((sum(nk), H, D), generator=g) for _ in range(2))
    cu_q, cu_k = (np.concatenate([[0], np.cumsum(n)]).astype(np.int32) for n in (nq, nk))
    q64, k64, v64, dA64 = (P.to64(t) for t in (q, k, v, dA))
    lists = (np.arange(sum(nq)), cu_q, np.arange(sum(nk)), cu_k, D ** -0.5)
    A, lse = sto.varlen_attention(q64, k64, v64, *lists)
    refs = sto.varlen_attention_bwd(q64, k64, v64, dA64, *lists)
    hat = lambda t: t.permute(1, 0, 2).contiguous().cuda()
    cq, ck = torch.from_numpy(cu_q).cuda(), torch.from_numpy(cu_k).cuda()
    oh, lse_g = mg.moga_varlen_attn_fwd(hat(q), hat(k), hat(v), cq, ck, D ** -0.5)
    P.assert_close_f32(P.unhat(oh), A, "O")
    fin = np.isfinite(lse)
    np.testing.assert_allclose(P.to64(lse_g).T[fin], lse[fin], rtol=1e-5, atol=1e-5)
    grads = mg.moga_varlen_attn_bwd(hat(dA), hat(q), hat(k), hat(v), oh, lse_g, cq, ck, D ** -0.5)
    for name, got, ref in zip(("dQ", "dK", "dV"), grads, refs):
        P.assert_close_f32(P.unhat(got), ref, name)
