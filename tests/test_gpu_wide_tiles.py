"""The large bf16 kernels at the edges of their tiles: last tiles of a group that take three columns of 16 rows per wave, two, or
leave waves idle, with either number of query rows and of keys per block, in pieces and whole, against the oracle with the tolerances
of the other bf16 cases."""
import numpy as np
import pytest
import torch

from oracle import moga_oracle as orc
from paper_2510_18692_amd import binding as mg
from tests import parity as P
from tests import test_gpu_backward as tb
from tests import test_gpu_forward as tf

pytestmark = pytest.mark.gpu

SIZES = [1, 47, 48, 49, 95, 97, 127, 128, 129, 255, 256, 257, 383, 384, 385, 639, 640, 641, 767, 769]


# in pieces, which is what the binding's workspace leads to for so few tiles
@pytest.mark.parametrize("H", [1, 2])
def test_forward_at_tile_edges(H):
    mg.set_small_group_rows(0)
    try:
        tf.test_group_attention_forward_matches_oracle(SIZES, H, 128, "bf16")
    finally:
        mg.set_small_group_rows(-1)


# in one launch, which the binding chooses for these, and apart in pieces; with the edges of 192-key tiles too
@pytest.mark.parametrize("pieces", [False, True], ids=["together", "pieces"])
@pytest.mark.parametrize("more", [[], [31, 33, 63, 65, 96, 143, 144, 145, 191, 192, 193, 320, 321]], ids=["rows", "rows and keys"])
def test_backward_at_tile_edges(more, pieces):
    sizes = SIZES + more
    mg.set_small_group_rows(0)
    try:
        if pieces:
            took, got, ref = backward_at_edges(sizes, 2, True)
            assert took[1] == took[3] == 1
            for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
                tb.check(P.unhat(a), b, name, "bf16")
        else:
            size = (sum(sizes), 2, 128, len(sizes), 0, mg.MOGA_BF16)
            ws = mg.load().moga_workspace_preferred_bytes(mg.OP_ATTN_BWD_JOINT, size[0], *size)
            assert mg.attn_blocks(mg.OP_ATTN_BWD_JOINT, size[0], size[0], 2, len(sizes), ws)[1] == 2
            tb.test_group_attention_backward_matches_oracle(sizes, 2, 128, "bf16")
    finally:
        mg.set_small_group_rows(-1)


# Heads with which either size of block is taken; 769 keys go round the ring of four 64-key tiles three times.  moga_group_attn_fwd has no
# room to split (every wave writes its finished rows), the others' workspace has.
@pytest.mark.parametrize("H,room,rows", [(1, False, 256), (5, False, 256), (7, False, 384), (9, False, 384), (1, True, 256), (10, True, 384)])
def test_forward_with_every_block_size(H, room, rows):
    print(f"H={H} room={room}", flush=True)
    q, k, v, cu, scale = tf.attn_case(SIZES, H, 128, "bf16", seed=H)
    A, lse = orc.group_attention(P.to64(q), P.to64(k), P.to64(v), cu, scale)
    N, M, lib = q.shape[0], len(SIZES), mg.load()
    mg.set_small_group_rows(0)
    try:
        size = lib.moga_workspace_preferred_bytes(mg.OP_ATTN_FWD, N, N, H, 128, M, 0, mg.MOGA_BF16) if room else 0
        assert mg.attn_blocks(mg.OP_ATTN_FWD, N, N, H, M, size)[:2] == (rows, room)
        hat = lambda t: t.permute(1, 0, 2).contiguous().cuda()
        qh, kh, vh, cu_d = hat(q), hat(k), hat(v), torch.from_numpy(cu).cuda()
        ws = torch.full((max(size, 16),), 0xFF, dtype=torch.uint8, device="cuda")
        oh, l = torch.empty_like(qh), torch.empty((H, N), device="cuda")
        fn = lib.moga_group_attn_fwd_ws if room else lib.moga_group_attn_fwd
        assert fn(qh.data_ptr(), kh.data_ptr(), vh.data_ptr(), mg.MOGA_BF16, N, H, 128, cu_d.data_ptr(), M, scale, oh.data_ptr(), l.data_ptr(),
                  ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
    finally:
        mg.set_small_group_rows(-1)
    P.assert_close_bf16(P.unhat(oh), A, "O")
    np.testing.assert_allclose(P.to64(l).T, lse, rtol=1e-3, atol=2e-3)


def backward_at_edges(sizes, H, room):
    """(dQ, dK, dV) and the oracle's, through the C entry with the workspace it needs (nothing is split) or with the preferred one."""
    q, k, v, dA, cu, scale = tb.attn_bwd_case(sizes, H, 128, "bf16", seed=H)
    q64, k64, v64, dA64 = (P.to64(t) for t in (q, k, v, dA))
    A, lse = orc.group_attention(q64, k64, v64, cu, scale)
    N, M = q.shape[0], len(sizes)
    lib = mg.load()
    need = mg.workspace_bytes(mg.OP_ATTN_BWD, N, H, 128, M, 0, mg.MOGA_BF16)
    size = lib.moga_workspace_preferred_bytes(mg.OP_ATTN_BWD, N, N, H, 128, M, 0, mg.MOGA_BF16) if room else need
    ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN wherever nothing is written
    hat = lambda t: t.permute(1, 0, 2).contiguous().cuda()
    oh, lse_d = torch.from_numpy(P.hat(A)).bfloat16().cuda(), torch.from_numpy(np.ascontiguousarray(lse.T)).float().cuda()
    got = mg.moga_group_attn_bwd(hat(dA), hat(q), hat(k), hat(v), oh, lse_d, torch.from_numpy(cu).cuda(), scale, ws=ws)
    torch.cuda.synchronize()
    assert int(mg.attn_bwd_status(ws, N, H).item()) == 0
    return mg.attn_blocks(mg.OP_ATTN_BWD, N, N, H, M, size), got, orc.group_attention_bwd(q64, k64, v64, dA64, cu, scale)


# Heads with which every pair of block sizes is taken; groups of up to 769 rows go round the ring of four 64-row tiles three times.
@pytest.mark.parametrize("H,room,blocks", [
    (1, False, (256, False, 128, False)), (5, False, (256, False, 192, False)), (7, False, (384, False, 128, False)),
    (9, False, (384, False, 192, False)), (1, True, (256, True, 128, True)), (10, True, (384, True, 192, True))])
def test_backward_with_every_block_size(H, room, blocks):
    print(f"H={H} room={room}", flush=True)
    mg.set_small_group_rows(0)
    try:
        took, got, ref = backward_at_edges(SIZES, H, room)
    finally:
        mg.set_small_group_rows(-1)
    print(took, flush=True)
    assert took == blocks
    for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
        tb.check(P.unhat(a), b, name, "bf16")


# token-order rows gathered by the kernels: forward blocks of either size that do not split; backward in one launch (both forms:
# test_gpu_fused_forms.py)
@pytest.mark.parametrize("H", [1, 5, 7, 9])
def test_gather_fused_calls_with_every_block_size(H):
    print(f"fused H={H}", flush=True)
    q, k, v, d_o, cu, scale = tb.attn_bwd_case(SIZES, H, 128, "bf16", seed=H + 20)   # sorted order
    N = q.shape[0]
    g = torch.Generator().manual_seed(H)
    perm, gate = torch.randperm(N, generator=g), torch.rand(N, generator=g) * 0.7 + 0.2
    tok = lambda t: torch.empty_like(t).index_copy_(0, perm, t)   # row j of the sorted order is token perm[j]
    gs = P.to64(gate)[perm.numpy()][:, None, None]
    q64, k64, v64, d64 = (P.to64(t) for t in (q, k, v, d_o))
    A, lse = orc.group_attention(q64, k64, v64, cu, scale)
    ref = orc.group_attention_bwd(q64, k64, v64, d64 * gs, cu, scale)
    o = tok(torch.from_numpy(A * gs).bfloat16()).cuda()
    inv = torch.empty(N, dtype=torch.int32)
    inv[perm] = torch.arange(N, dtype=torch.int32)
    o_got, lse_got = mg.moga_fused_attn_fwd(*(tok(t).cuda() for t in (q, k, v)), perm.int().cuda(), gate.cuda(), torch.from_numpy(cu).cuda(), scale)
    P.assert_close_bf16(P.to64(o_got.cpu()[perm]), A * gs, "O")
    np.testing.assert_allclose(P.to64(lse_got).T, lse, rtol=1e-3, atol=2e-3)
    *got, d_gate = mg.moga_fused_attn_bwd(*(tok(t).cuda() for t in (d_o, q, k, v)), o, torch.from_numpy(np.ascontiguousarray(lse.T)).float().cuda(),
                                          perm.int().cuda(), inv.cuda(), gate.cuda(), torch.from_numpy(cu).cuda(), scale)
    torch.cuda.synchronize()
    for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
        tb.check(P.to64(a.cpu()[perm]), b, name, "bf16")
    d_ref = np.empty(N)
    d_ref[perm.numpy()] = (d64 * A).sum(axis=(1, 2))
    np.testing.assert_allclose(P.to64(d_gate), d_ref, rtol=3e-2, atol=3e-2 * np.abs(d_ref).max())
