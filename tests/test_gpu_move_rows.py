"""Kernels that move rows: four tokens per block and sixteen, heads that do not fill a wave's four, tokens with any number of slots."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


def close(got, want, size, terms):
    """`got` is `want` rounded to its type after fp32 sums of `terms` terms of absolute values `size` altogether."""
    eps = 2.0 ** -8 if got.dtype == torch.bfloat16 else 2.0 ** -24
    assert bool(((got.double() - want).abs() <= eps * want.abs() + (terms + 2) * 2.0 ** -24 * size + 1e-37).all())


@pytest.mark.parametrize("N,H,D,dtype", [(1, 1, 128, "bf16"), (3, 5, 128, "bf16"), (5, 17, 128, "bf16"), (330, 12, 128, "bf16"), (67, 3, 64, "f32"),
                                         (33, 6, 128, "f32")])
def test_gradients_of_three_branches_in_one_launch(N, H, D, dtype):
    g = torch.Generator().manual_seed(N + H)
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    lists = torch.randint(0, 6, (N,), generator=g)   # slots of a token: none to five
    Nk = int(lists.sum())
    inv_cu = torch.cat([torch.zeros(1, dtype=torch.long), lists.cumsum(0)]).int().cuda()
    slot = torch.randperm(Nk, generator=g)
    slots = torch.cat([s.sort().values for s in slot.split(lists.tolist())] + [slot[:0]]).int().cuda()
    inv_m, q_slot, inv_f = (torch.randperm(N, generator=g).int().cuda() for _ in range(3))
    rnd = lambda n: torch.randn(H, n, D, generator=g).to(tt).cuda()
    m, f = [[rnd(N) for _ in range(3)] for _ in range(2)]
    s = [rnd(N), rnd(Nk), rnd(Nk)]
    ident = torch.arange(N + 1, dtype=torch.int32, device="cuda")
    for frame in (None, inv_f):
        got = mg.moga_gather3_bwd_qkv(m, inv_m, s, q_slot, inv_cu, slots, f, frame)
        for i in range(3):
            cu, sl = (ident, q_slot) if i == 0 else (inv_cu, slots)
            one = mg.moga_gather3_bwd(m[i], inv_m, s[i], cu, sl, f[i], frame)
            assert torch.equal(got[i], one)
            at = lambda t, idx: t[:, idx.long()].double().transpose(0, 1)
            of = torch.repeat_interleave(torch.arange(N, device="cuda"), cu.diff().long())
            terms = [at(m[i], inv_m), at(f[i], frame if frame is not None else ident[:N])]
            rows = at(s[i], sl)
            want = (terms[0] + terms[1]).index_add_(0, of, rows)
            size = (terms[0].abs() + terms[1].abs()).index_add_(0, of, rows.abs())
            close(one, want, size, 7)


@pytest.mark.parametrize("N,H", [(2, 1), (7, 6), (250, 13), (6000, 3), (6001, 3), (6007, 5)])   # 6,000: the last call with four tokens per block
def test_scatter_backward_and_its_sums(N, H):
    g = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *n: torch.randn(*n, generator=g, device="cuda")
    d_o, oh = rnd(N, H, 128).bfloat16(), rnd(H, N, 128).bfloat16()
    perm = torch.randperm(N, generator=g, device="cuda").int()
    gate = rnd(N).abs() + 0.1
    d_oh, d_gate = mg.moga_unpermute_bwd(d_o, oh, perm, gate)
    rows = d_o[perm.long()].double()
    gated = gate[perm.long()].double()[:, None, None] * rows
    close(d_oh, gated.transpose(0, 1), gated.abs().transpose(0, 1), 0)
    prod = rows * oh.transpose(0, 1).double()
    want, size = torch.zeros(2, N, dtype=torch.double, device="cuda")
    want[perm.long()], size[perm.long()] = prod.sum((1, 2)), prod.abs().sum((1, 2))
    close(d_gate, want, size, 8 * ((H + 3) // 4) + 8)   # a lane's eight products of every fourth head, 16 lanes, four waves
    o = mg.moga_unpermute(oh, perm, gate)
    back = torch.empty_like(o, dtype=torch.double)
    back[perm.long()] = oh.transpose(0, 1).double() * gate[perm.long()].double()[:, None, None]
    close(o, back, back.abs(), 0)
    inv = torch.empty_like(perm)
    inv[perm.long()] = torch.arange(N, dtype=torch.int32, device="cuda")
    a_s, a_f = rnd(H, N, 128).bfloat16(), rnd(H, N, 128).bfloat16()
    d_m, d_s, d_f, d_g = mg.moga_merge3_bwd(d_o, oh, inv, None, None, gate)
    third = (gate * (1 / 3)).double()[perm.long()][:, None, None]
    close(d_m, (third * rows).transpose(0, 1), (third * rows.abs()).transpose(0, 1), 2)
    close(d_g, want / 3, size / 3, 8 * ((H + 3) // 4) + 10)
    assert torch.equal(d_s, d_f)
    mean = mg.moga_merge3_fwd(oh, a_s, a_f, inv, None, None, gate)
    want3 = (gate.double()[:, None, None] * oh.transpose(0, 1)[inv.long()].double() + a_s.transpose(0, 1).double() + a_f.transpose(0, 1).double()) / 3
    size3 = (gate.double()[:, None, None] * oh.transpose(0, 1)[inv.long()].double().abs() + a_s.transpose(0, 1).double().abs()
             + a_f.transpose(0, 1).double().abs()) / 3
    close(mean, want3, size3, 4)
