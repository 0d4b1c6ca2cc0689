"""The torch.autograd wrapper returns the oracle's gradients (it only chains the C-ABI calls)."""
import numpy as np
import pytest
import torch

from oracle import moga_oracle as orc
from paper_2510_18692_amd import binding as mg
from paper_2510_18692_amd import workloads as wl
from paper_2510_18692_amd.autograd import moga_attention
from tests import parity as P

pytestmark = pytest.mark.gpu


def test_autograd_gradients_match_oracle_with_balancing_loss():
    w = wl.WORKLOADS["C1b"]
    inp = wl.make_inputs(w, "cpu")
    X, W, Q, K, V, dO = (P.to64(inp[k]) for k in ("X", "W", "Q", "K", "V", "dO"))
    alpha, lam = 0.1, 3.0                      # total loss = sum(O * dO) + lam * L_balance
    f = orc.moga_forward(X, W, Q, K, V, w.scale)
    b = orc.moga_backward(f, X, W, dO, w.scale)
    d_gate = b["d_gate"] + lam * orc.balance_loss_bwd(f["group"], w.M, alpha)
    dW, dX, _ = orc.route_bwd(X, W, f["probs"], f["group"], f["gate"], d_gate, want_dx=True)
    t = {k: inp[k].cuda().requires_grad_(k != "dO") for k in ("X", "W", "Q", "K", "V", "dO")}
    o, lb, group = moga_attention(t["X"], t["W"], t["Q"], t["K"], t["V"], w.scale, balance_alpha=alpha, grad_x=True)
    assert not P.check_assignment(group.cpu().numpy(), f)
    ((o * t["dO"]).sum() + lam * lb).backward()
    torch.cuda.synchronize()
    np.testing.assert_allclose(float(lb.item()), orc.balance_loss(f["group"], f["gate"], w.M, alpha)[0], rtol=1e-5)
    P.assert_close_f32(P.to64(o.detach()), f["O"], "O")
    for name, ref in (("Q", b["dQ"]), ("K", b["dK"]), ("V", b["dV"]), ("W", dW), ("X", dX)):
        e = P.assert_close_f32(P.to64(t[name].grad), ref, "d" + name)
        print(f"  d{name} rel err {e:.2e}", flush=True)


# bf16 with the balancing loss and d_x, against the separate calls bit by bit: few rows, all in the pass's one allocation; d_oh above 64 MiB, in one
# of its own; an attention backward that is given room to split a round; groups that do not fill their parts; fp32 of head_dim 128
@pytest.mark.parametrize("N,H,D,d_model,M,dtype,own_rows,own_ws", [
    (1560, 4, 128, 512, 8, "bf16", False, False), (333, 3, 128, 256, 5, "bf16", False, False), (22000, 12, 128, 256, 16, "bf16", True, False),
    (8000, 3, 128, 256, 1, "bf16", False, True), (24325, 12, 128, 512, 2, "bf16", True, True), (700, 2, 128, 64, 3, "f32", False, False),
])
def test_autograd_is_the_separate_calls(N, H, D, d_model, M, dtype, own_rows, own_ws):
    print(f"autograd N={N} H={H} {dtype}", flush=True)
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    if dtype == "bf16":
        size = (N, H, D, M, 0, mg.MOGA_BF16)
        assert (mg.load().moga_workspace_preferred_bytes(mg.OP_ATTN_BWD_JOINT, N, *size) > mg.workspace_bytes(mg.OP_ATTN_BWD_JOINT, *size)) == own_ws
    assert (N * H * D * tt.itemsize > 64 << 20) == own_rows
    g = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *n: torch.randn(n, generator=g, device="cuda")
    x, q, k, v, d_o = (rnd(*n).to(tt) for n in [(N, d_model)] + [(N, H, D)] * 4)
    w, alpha, lam = rnd(M, d_model) * 0.2, 0.1, torch.tensor(2.5, device="cuda")
    scale = D ** -0.5

    group, gate, probs, _ = mg.moga_route(x, w)
    pm = mg.moga_permute(group, M, q, k, v)
    oh, lse = mg.moga_group_attn_fwd(pm["qh"], pm["kh"], pm["vh"], pm["cu_seqlens"], scale)
    o = mg.moga_unpermute(oh, pm["perm"], gate)
    loss, frac, _ = mg.moga_balance_loss(group, gate, M, alpha)
    d_oh, d_gate = mg.moga_unpermute_bwd(d_o, oh, pm["perm"], gate)
    rows = mg.moga_group_attn_bwd(d_oh, pm["qh"], pm["kh"], pm["vh"], oh, lse, pm["cu_seqlens"], scale)
    want = [*mg.moga_permute_bwd(*rows, pm["perm"])]
    d_w, d_x = mg.moga_route_bwd_balanced(x, w, probs, group, gate, d_gate, frac, alpha, lam, want_dx=True)
    want += [d_w, d_x.to(tt)]

    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    poison = [torch.full((n,), 255, dtype=torch.uint8, device="cuda") for n in (1 << 28, 1 << 24, 1 << 19, 1 << 19, 4096, 4096)]
    del poison   # NaN wherever a part of an allocation is read before it is written
    t = [a.clone().requires_grad_() for a in (q, k, v, w, x)]
    o_a, loss_a, group_a = moga_attention(t[4], t[3], *t[:3], scale, balance_alpha=alpha, grad_x=True)
    grads = torch.autograd.grad([o_a, loss_a], t, [d_o, lam])
    assert torch.equal(o_a, o) and torch.equal(group_a, group) and torch.equal(loss_a.reshape(1), loss.reshape(1))
    for a, b in zip(grads, want):
        assert a.dtype == b.dtype and torch.equal(a, b)
