"""Several attention calls in one launch against float64 attention of each, with either set of kernels and either size of block."""
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


def reference(q, k, v, d_o, cu_q, cu_k, scale):
    """(o, d_q, d_k, d_v) in float64; [H, N, D] each."""
    q, k, v = (t.double().requires_grad_(True) for t in (q, k, v))
    o = 0 * q
    for a, b, c, d in zip(cu_q, cu_q[1:], cu_k, cu_k[1:]):
        if b > a and d > c:
            p = torch.softmax(scale * (q[:, a:b] @ k[:, c:d].transpose(1, 2).contiguous()), dim=2)
            o = torch.cat([o[:, :a], p @ v[:, c:d], o[:, b:]], dim=1)
    grads = torch.autograd.grad(o, (q, k, v), d_o.double(), allow_unused=True)
    return [o.detach()] + [torch.zeros_like(t) if g is None else g for g, t in zip(grads, (q, k, v))]


def sums(sizes):
    return torch.tensor([0, *sizes]).cumsum(0).tolist()


# (queries, keys) of the groups of each call: empty groups, groups without keys or without queries, ends inside a tile, more than 256 groups (the
# tiles are summed by a kernel of their own), one call, calls without queries; "wide" has blocks of 384 queries and 192 keys, "many
# rounds" (64 heads) dQ and dK/dV of all calls in a launch each
CALLS = {
    "mixed": [([700, 0, 33, 385], [700, 0, 33, 385]), ([130, 64, 1], [300, 0, 65]), ([100, 100], [7, 129])],
    "many groups": [([3] * 300, [5] * 300), ([1000], [900])],
    "one": [([200, 100], [100, 90])],
    "no queries": [([0, 0], [10, 20]), ([40], [50]), ([300], [300])],
    "many rounds": [([1024] * 8, [1000] * 8), ([1024, 1100, 500], [1024, 1100, 0]), ([2000], [2])],
    "windows": [([1000, 0, 930], [1000, 0, 930]), ([16] * 120 + [9], [16] * 120 + [23]), ([640] * 3, [640] * 3)],   # 1.06 rounds with 12 heads
    "long": [([8300], [8300]), ([130] * 10, [150] * 10), ([700, 900], [700, 900])],   # the first by itself, its last round split
    "wide": [([1536] * 4, [1536] * 4), ([384, 100, 500], [700, 200, 193]), ([1000], [1001])],
}


CASES = [(name, rows, torch.bfloat16) for name in CALLS for rows in (-1, 0, 1 << 40)] + [("mixed", -1, torch.float32)]   # fp32: one after the other


@pytest.mark.parametrize("name,small_rows,dtype", CASES)
def test_calls_together(name, small_rows, dtype):
    H, D = {"wide": 16, "many rounds": 64, "windows": 12}.get(name, 3), 128
    gen = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda n: torch.randn((H, n, D), generator=gen, device="cuda").to(dtype)
    scale, shapes = D ** -0.5, CALLS[name]
    calls = [(rnd(sum(q)), rnd(sum(k)), rnd(sum(k)), rnd(sum(q)), sums(q), sums(k)) for q, k in shapes]
    dev = lambda t: torch.tensor(t, dtype=torch.int32, device="cuda")
    rel = 1e-2 if dtype == torch.bfloat16 else 5e-6
    try:
        mg.set_small_group_rows(small_rows)
        fwd = mg.moga_varlen_attn_fwd_calls([(q, k, v, dev(cq), dev(ck)) for q, k, v, _, cq, ck in calls], scale)
        bwd_in = []
        for (q, k, v, d_o, cq, ck), (oh, lse) in zip(calls, fwd):
            n = q.shape[1] * H   # row constants as moga_merge3_bwd_rows leaves them: -delta, -lse / scale, status word
            need = mg.workspace_bytes(mg.OP_VARLEN_ATTN_BWD, q.shape[1], H, D, len(cq) - 1, 0, mg.MOGA_BF16)
            ws = torch.zeros(max(16, need), dtype=torch.uint8, device="cuda")
            f = ws[:8 * n].view(torch.float32)
            f[:n] = -(d_o.float() * oh.float()).sum(2).flatten()
            f[n:2 * n] = -lse.flatten() / scale
            bwd_in.append((d_o, q, k, v, oh, lse, dev(cq), dev(ck), ws))
        bwd = mg.moga_varlen_attn_bwd_rows_calls(bwd_in, scale)
        single = [mg.moga_varlen_attn_bwd_rows(*c[:8], scale, c[8]) for c in bwd_in]
    finally:
        mg.set_small_group_rows(-1)
    for (q, k, v, d_o, cq, ck), (oh, lse), grads, alone, c in zip(calls, fwd, bwd, single, bwd_in):
        want = reference(q, k, v, d_o, cq, ck, scale)
        for got, w in zip([oh, *grads], want):
            assert got.shape == w.shape
            assert not torch.isnan(got).any()
            assert (got.double() - w).norm() <= rel * w.norm()
        for got, w in zip(grads, alone):   # other blocks, other order of the sums
            assert (got.double() - w.double()).norm() <= rel * w.double().norm()
        assert int(c[8][8 * q.shape[1] * H:].view(torch.int32)[0] if q.shape[1] else 0) == 0   # no wave gave up


# one launch for dQ and dK/dV against the two of the call with a workspace of its own: no round is split, so only the small-group kernels and
# the large ones differ in their bits.  The tiles of the first product end before, at and after the blocks that it has for sure, and far before
# those that the host counts (empty groups)
@pytest.mark.parametrize("sizes,H", [([300, 0, 77], 3), ([1], 1), ([900, 1300, 2100, 5], 4), ([640] * 9, 12), ([1536] * 4, 16), ([3000], 1),
                                     ([1536] + [0] * 60, 14), ([0] * 70 + [1, 129, 257] + [0] * 30, 3), ([1] * 255 + [900], 1), ([2048], 8)])
@pytest.mark.parametrize("small_rows", [0, 1 << 40])
def test_one_launch_gives_the_bits_of_two(sizes, H, small_rows):
    gen = torch.Generator(device="cuda").manual_seed(H)
    q, k, v, d_o = (torch.randn((H, sum(sizes), 128), generator=gen, device="cuda").bfloat16() for _ in range(4))
    cu, scale = torch.tensor(sums(sizes), dtype=torch.int32, device="cuda"), 128 ** -0.5
    need = mg.workspace_bytes(mg.OP_ATTN_BWD_JOINT, q.shape[1], H, 128, len(sizes), 0, mg.MOGA_BF16)
    lib, stream = mg.load(), torch.cuda.current_stream().cuda_stream
    ptr = lambda *t: [x.data_ptr() for x in t]
    try:
        mg.set_small_group_rows(small_rows)
        oh, lse = mg.moga_group_attn_fwd(q, k, v, cu, scale)

        def run(fn):
            ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
            g = [torch.full_like(q, float("nan")) for _ in range(3)]
            assert fn(*ptr(d_o, q, k, v, oh, lse), mg.MOGA_BF16, q.shape[1], H, 128, cu.data_ptr(), len(sizes), scale, *ptr(*g, ws), need, stream) == 0
            torch.cuda.synchronize()
            return g, int(mg.attn_bwd_status(ws, q.shape[1], H))

        got, flag = run(lib.moga_group_attn_bwd_joint)
        want, _ = run(lib.moga_group_attn_bwd)
        assert flag == 0
        for x, y in zip(got, want):
            assert torch.equal(x, y)
        mg.set_spin_limit(0)
        assert run(lib.moga_group_attn_bwd_joint)[1] != 0   # the waits are bounded: every wave gave up, and the kernel drained
    finally:
        mg.set_spin_limit(1 << 24)
        mg.set_small_group_rows(-1)


def test_calls_that_are_refused():
    t = torch.zeros((2, 8, 128), device="cuda", dtype=torch.bfloat16)
    cu = torch.tensor([0, 8], dtype=torch.int32, device="cuda")
    ok = (t, t, t, cu, cu)
    with pytest.raises(RuntimeError):
        mg.moga_varlen_attn_fwd_calls([ok] * 4, 0.1)
    with pytest.raises(RuntimeError):
        mg.moga_varlen_attn_fwd_calls([], 0.1)
    with pytest.raises(RuntimeError):
        mg.moga_varlen_attn_fwd_calls([ok, (t[:1].contiguous(), t[:1].contiguous(), t[:1].contiguous(), cu, cu)], 0.1)
    with pytest.raises(mg.MogaError):
        mg.moga_varlen_attn_fwd_calls([ok, ok], float("inf"))
