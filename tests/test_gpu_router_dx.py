"""The router's gradient of its input: every launch shape of the kernel, as fp32 and rounded to bf16."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


# group words of 8, 16 and 32; columns by 8, by 4 (d no multiple of 8, more than 16 groups) and one at a time (d no multiple of 4, more
# than 32 groups); blocks of 64 to 256 threads, a column slab that is not full, several slabs; token tiles with a remainder
SHAPES = [(1, 4, 1), (15, 64, 8), (16, 512, 9), (33, 200, 5), (17, 516, 16), (1000, 1540, 17), (700, 2056, 32), (300, 100, 40),
          (64, 63, 3), (4100, 5120, 8), (9000, 1536, 5)]


@pytest.mark.parametrize("N,d,M", SHAPES)
@pytest.mark.parametrize("frac", [False, True])
def test_dx_of_either_type(N, d, M, frac):
    torch.manual_seed(N + d + M)
    x = torch.randn(N, d).cuda().bfloat16()
    w = torch.randn(M, d).cuda()
    p = torch.softmax(2 * torch.randn(N, M), dim=1).cuda()
    group = torch.randint(0, M, (N,), dtype=torch.int32).cuda()
    gate = p.gather(1, group[:, None].long())[:, 0].contiguous()
    d_gate = torch.randn(N).cuda()
    fr = torch.bincount(group.long(), minlength=M).float().div(N) if frac else None
    ws = torch.empty(max(16, mg.workspace_bytes(mg.OP_ROUTE_BWD, N, 0, 0, M, d, mg.MOGA_BF16)), dtype=torch.uint8, device="cuda")
    lib = mg.load()

    def dx(out, code):
        d_w = torch.empty(M, d, device="cuda")
        args = (x.data_ptr(), 1, w.data_ptr(), p.data_ptr(), group.data_ptr(), gate.data_ptr(), d_gate.data_ptr(),
                fr.data_ptr() if frac else None, 0.1, 1.0, None, N, d, M, d_w.data_ptr(), out.data_ptr(), code, ws.data_ptr(),
                ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert lib.moga_route_bwd_typed(*args) == 0
        torch.cuda.synchronize()
        return out.clone()

    f32 = dx(torch.full((N, d), float("nan"), device="cuda"), 0)
    coef = d_gate.double() + ((0.1 * M / N) * fr.double()[group.long()] if frac else 0.)
    dr = (coef * gate.double())[:, None] * (torch.nn.functional.one_hot(group.long(), M).double() - p.double())
    want = dr @ w.double()
    # M fmas and some five roundings of each factor
    bound = (M + 6) * 2.0 ** -24 * ((d_gate.abs().double() + (0.1 * M / N if frac else 0.))[:, None] * gate.double()[:, None]
                                    * (torch.nn.functional.one_hot(group.long(), M).double() + p.double()) @ w.abs().double())
    assert bool(((f32.double() - want).abs() <= bound + 1e-37).all())
    half = dx(torch.full((N, d), float("nan"), device="cuda", dtype=torch.bfloat16), 1)
    assert torch.equal(half, f32.bfloat16())
    # a start that only takes 8-byte stores
    odd = torch.full((N * d + 4,), float("nan"), device="cuda", dtype=torch.bfloat16)[4:]
    assert torch.equal(dx(odd, 1).view(N, d), half)
    code = lib.moga_route_bwd_typed(x.data_ptr(), 1, w.data_ptr(), p.data_ptr(), group.data_ptr(), gate.data_ptr(), d_gate.data_ptr(),
                                    None, 0.1, 1.0, None, N, d, M, ws.data_ptr(), half.data_ptr(), 7, ws.data_ptr(), ws.numel(), None)
    assert code != 0   # no such type
