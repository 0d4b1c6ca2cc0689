"""Calls given another stream than torch's current one: their workspaces and the results they drop are not handed to the
current stream while the kernels may still run.  The side stream is kept busy first, so that every call returns long before
its kernels start, and the current stream then allocates and overwrites all it can get of the sizes that were dropped."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg
from paper_2510_18692_amd import workloads as wl

pytestmark = pytest.mark.gpu


def grab():
    return [torch.full((1 << e,), 0x7F, dtype=torch.uint8, device="cuda") for e in range(9, 26) for _ in range(4)]


def on_busy_side_stream(fn):
    """fn(side) with the side stream asleep; its results once both streams are through."""
    side = torch.cuda.Stream()
    grab()   # memory for it is in torch's cache now: no allocation by the device below
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)   # a tenth of a second or more
    asleep = torch.cuda.Event()
    asleep.record(side)
    out = fn(side)
    keep = grab()
    assert not asleep.query(), "the side stream was not busy for long enough"
    torch.cuda.synchronize()
    del keep
    return out


def test_forward_backward_and_balance_loss():
    w = wl.scaled(wl.WORKLOADS["C5"], N=20000, H=4, d_model=512, M=8)   # permutation in three kernels, dW in splits
    i = wl.make_inputs(w, "cuda")
    half = torch.tensor(0.5, dtype=torch.float64, device="cuda")        # converted to float before the kernel reads it

    def step(stream):
        f = mg.moga_forward(i["X"], i["W"], i["Q"], i["K"], i["V"], w.scale, stream=stream)
        b = mg.moga_backward(f, i["X"], i["W"], i["dO"], w.scale, want_dx=True, stream=stream)
        loss, frac, _ = mg.moga_balance_loss(f["group"], f["gate"], w.M, 0.1, stream=stream)
        g = mg.moga_balance_loss_bwd(f["group"], frac, 0.1, d_loss=half, stream=stream)
        return [f[k] for k in ("perm", "inv_perm", "cu_seqlens", "lse", "o")] + [b[k] for k in ("d_q", "d_k", "d_v", "d_w", "d_x")] + [loss, g]

    mg.set_small_group_rows(1 << 40)   # no split last round on either stream: the same bits
    try:
        ref = step(None)
        got = on_busy_side_stream(step)
    finally:
        mg.set_small_group_rows(-1)
    for n, (a, b) in enumerate(zip(got, ref)):
        assert torch.equal(a, b), n


def test_three_branch_block():
    T, Hh, Ww, H, M = 4, 10, 18, 2, 4
    N = T * Hh * Ww
    g = torch.Generator().manual_seed(5)
    q, k, v, d_o = (torch.randn((N, H, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(4))
    x = torch.randn((N, 256), generator=g).to(torch.bfloat16).cuda()
    w = (torch.randn((M, 256), generator=g) / 16).cuda()
    si = mg.moga_stga_build_index(T, Hh, Ww, 5, 6, 2, [0, 0, 1, 1])

    def step(stream):   # the intermediate gradients are dropped inside, everything else on return
        f = mg.visual_forward(x, w, q, k, v, 128 ** -0.5, (T, Hh, Ww), si, stream=stream)
        b = mg.visual_backward(f, x, w, d_o, 128 ** -0.5, stream=stream)
        return [f["o"]] + [b[n] for n in ("d_q", "d_k", "d_v", "d_w")]

    ref = step(None)
    for n, (a, b) in enumerate(zip(on_busy_side_stream(step), ref)):
        assert torch.equal(a, b), n
