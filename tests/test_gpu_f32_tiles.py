"""fp32 attention kernels (32-row blocks, eight waves sharing the streamed rows) at the sizes where their
split can go wrong: around one step (32 rows), around one round of the eight waves (256 rows), sides without
rows, different query and key lists.  Against the float64 oracle, relative to the largest value: 1e-4, the
bound of the fp32 configuration (fp32 sums of at most 600 terms of a convex combination err by a few 1e-6)."""
import numpy as np
import pytest
import torch

from oracle import stga_oracle as sto
from paper_2510_18692_amd import binding as mg
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("nq,nk", [
    ([1, 31, 32, 33], [1, 31, 32, 33]),
    ([255, 256, 257], [255, 256, 257]),
    ([32, 0, 40, 7, 64], [289, 33, 0, 1, 600]),      # more and fewer keys than queries, empty sides
])
def test_f32_attention_tile_edges(D, nq, nk):
    print(f"f32 tiles D={D} nq={nq} nk={nk}", flush=True)
    H, scale = 2, D ** -0.5
    g = torch.Generator().manual_seed(D + sum(nq))
    Nq, Nk = sum(nq), sum(nk)
    q, dA = (torch.randn((Nq, H, D), generator=g) for _ in range(2))
    k, v = (torch.randn((Nk, H, D), generator=g) for _ in range(2))
    cu_q = np.concatenate([[0], np.cumsum(nq)]).astype(np.int32)
    cu_k = np.concatenate([[0], np.cumsum(nk)]).astype(np.int32)
    q64, k64, v64, dA64 = (P.to64(t) for t in (q, k, v, dA))
    A, lse = sto.varlen_attention(q64, k64, v64, np.arange(Nq), cu_q, np.arange(Nk), cu_k, scale)
    refs = sto.varlen_attention_bwd(q64, k64, v64, dA64, np.arange(Nq), cu_q, np.arange(Nk), cu_k, scale)
    hat = lambda t: t.permute(1, 0, 2).contiguous().cuda()
    cq, ck = torch.from_numpy(cu_q).cuda(), torch.from_numpy(cu_k).cuda()
    oh, lse_g = mg.moga_varlen_attn_fwd(hat(q), hat(k), hat(v), cq, ck, scale)
    P.assert_close_f32(P.unhat(oh), A, "O")
    fin = np.isfinite(lse)
    np.testing.assert_allclose(P.to64(lse_g).T[fin], lse[fin], rtol=1e-5, atol=1e-5)
    assert np.all(np.isneginf(P.to64(lse_g).T[~fin]))
    grads = mg.moga_varlen_attn_bwd(hat(dA), hat(q), hat(k), hat(v), oh, lse_g, cq, ck, scale)
    torch.cuda.synchronize()
    for name, got, ref in zip(("dQ", "dK", "dV"), grads, refs):
        P.assert_close_f32(P.unhat(got), ref, name)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("first,count", [(0, 32), (32, 32), (5, 300), (224, 76)])
def test_f32_keys_with_scores_of_minus_infinity_have_no_weight(D, first, count):
    """A run of keys so large that their scores overflow to -inf (whole steps of a wave, the first ones among them):
    the rows equal those without these keys.  Group of 300 queries and 700 keys, every query entry positive."""
    g = torch.Generator().manual_seed(D + first)
    q, k, v = torch.rand((2, 300, D), generator=g) + 0.5, torch.randn((2, 700, D), generator=g), torch.randn((2, 700, D), generator=g)
    keep = torch.ones(700, dtype=torch.bool)
    keep[first:first + count] = False
    k[:, ~keep] = -3e38
    cq = torch.tensor([0, 300], dtype=torch.int32, device="cuda")
    out = []
    for kk, vv in ((k, v), (k[:, keep], v[:, keep])):
        ck = torch.tensor([0, kk.shape[1]], dtype=torch.int32, device="cuda")
        out.append(mg.moga_varlen_attn_fwd(q.cuda(), kk.contiguous().cuda(), vv.contiguous().cuda(), cq, ck, D ** -0.5))
    for a, b, name in zip(out[0], out[1], ("O", "lse")):
        P.assert_close_f32(P.to64(a), P.to64(b), name)


@pytest.mark.parametrize("D", [64, 128])
def test_f32_infinity_in_the_last_row_of_a_group(D):
    """Groups that end inside a step (33 and 300 rows): an infinite entry of V in the last row makes its channel of O
    infinite, one of dO its channel of dV, and nothing there NaN."""
    g = torch.Generator().manual_seed(D)
    q, k, v, d = (torch.randn((1, 333, D), generator=g) for _ in range(4))
    cu = torch.tensor([0, 33, 333], dtype=torch.int32, device="cuda")
    hv, hd = v.clone(), d.clone()
    for row in (32, 332):
        hv[0, row, 7] = hd[0, row, 7] = torch.inf
    q, k, v, d, hv, hd = (t.cuda() for t in (q, k, v, d, hv, hd))
    o, _ = mg.moga_group_attn_fwd(q, k, hv, cu, D ** -0.5)
    o0, lse = mg.moga_group_attn_fwd(q, k, v, cu, D ** -0.5)
    dv = mg.moga_group_attn_bwd(hd, q, k, v, o0, lse, cu, D ** -0.5)[2]
    dv0 = mg.moga_group_attn_bwd(d, q, k, v, o0, lse, cu, D ** -0.5)[2]
    for a, b in ((o, o0), (dv, dv0)):
        a, b = a.cpu(), b.cpu()
        assert (a[..., 7] == torch.inf).all()
        assert torch.equal(a[..., :7], b[..., :7]) and torch.equal(a[..., 8:], b[..., 8:])


def test_f32_backward_probabilities_keep_their_precision_at_large_logits():
    """P = exp(scale s - lse) of the backward, read off the gradients: dot products that are exact in fp32, dO = unit rows
    (dV = P^T), V = ones and O = 0 (dS = P, which dQ and dK show in channels of their own).  With x = scale s - lse rounded
    once, times log2(e), and exp2 good to two units, P is off by at most (2.3 |x| + 8) 2^-24 of itself; logits are
    64 to 136 here, and anything rounded at their size shows (100 * 2^-24 = 6e-6 against 5e-7 to 2e-6)."""
    D, nq, nk, scale = 64, 31, 32, float(np.float32(0.1))
    a, b = 32.0 + np.arange(nq), (20.0 + np.arange(nk) / 16.0)
    q, k, d = np.zeros((nq, D)), np.zeros((nk, D)), np.zeros((nq, D))
    q[:, 0], k[:, 0] = a, b
    k[np.arange(nk), 1 + np.arange(nk)] = 1.0               # channels 1 .. 32: a key each
    q[np.arange(nq), 33 + np.arange(nq)] = 1.0              # channels 33 .. 63: a query each
    d[np.arange(nq), np.arange(nq)] = 1.0
    logits = scale * np.outer(a, b)
    lse = (logits.max(1) + 0.5).astype(np.float32)
    x = logits - lse.astype(np.float64)[:, None]
    assert logits.max() > 100 and -16 < x.min() and x.max() < 0
    f = lambda t: torch.from_numpy(t.astype(np.float32))[None].cuda()
    cu = lambda n: torch.tensor([0, n], dtype=torch.int32, device="cuda")
    dq, dk, dv = mg.moga_varlen_attn_bwd(f(d), f(q), f(k), torch.ones((1, nk, D), device="cuda"), torch.zeros((1, nq, D), device="cuda"),
                                         f(lse), cu(nq), cu(nk), scale)
    bound = (2.3 * np.abs(x) + 8) * 2.0 ** -24
    for name, got in (("dV", P.to64(dv)[0][:, :nq].T), ("dQ", P.to64(dq)[0][:, 1:33] / scale), ("dK", P.to64(dk)[0][:, 33:].T / scale)):
        e = np.abs(got / np.exp(x) - 1)
        print(f"  {name}: largest error {e.max():.2e}, {(e / bound).max():.2f} of its bound", flush=True)
        assert (e <= bound).all(), name
