"""The native half of the binding: errors reach Python as before (CPU), and the native autograd function handles
outputs that do not take part in the loss (GPU)."""
import os

import numpy as np
import pytest
import torch

from paper_2510_18692_amd import binding as mg
from paper_2510_18692_amd import build
from paper_2510_18692_amd import workloads as wl
from paper_2510_18692_amd.autograd import moga_attention


def test_host_tensors_are_refused():
    x, w = torch.zeros(8, 64), torch.zeros(4, 64)
    with pytest.raises(AssertionError):
        mg.moga_route(x, w)
    with pytest.raises(AssertionError):
        mg.moga_permute(torch.zeros(8, dtype=torch.int32), 4)


def test_native_module_belongs_to_one_torch(monkeypatch):
    """Another torch in the same tree does not load the module built for this one: it asks for a build of its own."""
    path = build.native_path()
    mg._load_native()
    assert os.path.exists(path)
    built = []

    class Asked(Exception):
        pass

    def no_compiler():
        built.append(build.native_path())
        raise Asked

    monkeypatch.setattr(build, "build_native", no_compiler)
    mg._load_native()   # there already
    monkeypatch.setattr(torch, "__version__", "0.0.1+other")
    with pytest.raises(Asked):
        mg._load_native()
    assert built and built[0] != path


@pytest.mark.gpu
def test_status_codes_and_layout_errors_raise():
    x, w = torch.zeros(8, 64).cuda(), torch.zeros(300, 64).cuda()
    # not `as e`: the exception would keep this frame and its tensors until the next collection of cycles, which the
    # memory counts of other tests may see
    with pytest.raises(mg.MogaError, match=r"MOGA_ERR_UNSUPPORTED \(-2\)"):
        mg.moga_route(x, w)
    with pytest.raises(AssertionError):
        mg.moga_route(torch.zeros(64, 8).cuda().t(), w[:4])
    with pytest.raises(TypeError):
        mg.moga_gather_rows(torch.zeros(8, 2, 64, dtype=torch.float64).cuda(), torch.zeros(3, dtype=torch.int32).cuda())
    with pytest.raises(ValueError):
        mg.moga_route(torch.zeros(64).cuda(), w[:4])


@pytest.mark.gpu
@pytest.mark.parametrize("use", ["output", "loss", "both"])
def test_autograd_with_unused_outputs(use):
    w = wl.scaled(wl.WORKLOADS["C1b"], N=300)
    inp = wl.make_inputs(w, "cuda")
    t = {k: inp[k].clone().requires_grad_() for k in ("W", "Q", "K", "V")}
    o, lb, _ = moga_attention(inp["X"], t["W"], t["Q"], t["K"], t["V"], w.scale, balance_alpha=0.1)
    if use == "both":
        ((o * inp["dO"]).sum() + lb * 2.0).backward()
    else:
        ((o * inp["dO"]).sum() if use == "output" else lb * 2.0).backward()
    # the same gradients from the single calls
    f = mg.moga_forward(inp["X"], inp["W"], inp["Q"], inp["K"], inp["V"], w.scale)
    d_o = inp["dO"] if use != "loss" else torch.zeros_like(inp["dO"])
    d_oh, d_gate = mg.moga_unpermute_bwd(d_o, f["oh"], f["perm"], f["gate"])
    if use != "output":
        _, frac, _ = mg.moga_balance_loss(f["group"], f["gate"], w.M, 0.1)
        mg.moga_balance_loss_bwd(f["group"], frac, 0.1, d_loss=2.0, d_gate=d_gate)
    hats = mg.moga_group_attn_bwd(d_oh, f["qh"], f["kh"], f["vh"], f["oh"], f["lse"], f["cu_seqlens"], w.scale)
    ref = dict(zip("QKV", mg.moga_permute_bwd(*hats, f["perm"])))
    ref["W"], _ = mg.moga_route_bwd(inp["X"], inp["W"], f["probs"], f["group"], f["gate"], d_gate)
    torch.cuda.synchronize()
    for k, r in ref.items():
        assert np.array_equal(t[k].grad.cpu().numpy(), r.cpu().numpy()), k


@pytest.mark.gpu
@pytest.mark.parametrize("grad_x", [False, True])
def test_autograd_without_the_balancing_loss(grad_x):
    w = wl.scaled(wl.WORKLOADS["C1b"], N=300)
    inp = wl.make_inputs(w, "cuda")
    t = {k: inp[k].clone().requires_grad_() for k in ("X", "W", "Q", "K", "V")}
    o, loss, group = moga_attention(t["X"], t["W"], t["Q"], t["K"], t["V"], w.scale, grad_x=grad_x)
    assert loss is None and not group.requires_grad
    (o * inp["dO"]).sum().backward()
    f = mg.moga_forward(inp["X"], inp["W"], inp["Q"], inp["K"], inp["V"], w.scale)
    b = mg.moga_backward(f, inp["X"], inp["W"], inp["dO"], w.scale, want_dx=grad_x)
    torch.cuda.synchronize()
    assert torch.equal(o, f["o"]) and torch.equal(group, f["group"])
    for k, r in (("W", "d_w"), ("Q", "d_q"), ("K", "d_k"), ("V", "d_v")):
        assert torch.equal(t[k].grad, b[r]), k
    if grad_x:
        assert torch.equal(t["X"].grad, b["d_x"].to(t["X"].dtype))
    else:
        assert t["X"].grad is None
