"""Attention calls that split their last round against the same calls without room for it: numbers of tiles around the
edges of the rule (256 blocks a round, at most 8 pieces a tile), groups with fewer keys than pieces, and no keys at all.

Both ways round P and dS to bf16 (2^-9 relative at most, relative to another maximum per piece in the forward) and the
results once: 2-norms differ by less than 4 * 2^-9.  1e-5: where dP - delta cancels, fp32 rounding is left.  Row by row:
gradients differ by their own rounding alone (P and dS do not depend on the split), 2 * 2^-9 of a row; O by the rounding of
P too, whose share of a row of few keys or cancelling values is larger: 16 * 2^-9 (a row that is wrong is off by all of it);
lse by the rounded P that it sums, 2 * 2^-9 absolute at most."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2510_18692_amd import binding as mg

pytestmark = pytest.mark.gpu


def p(t):
    return t.data_ptr()


def close(a, b, name):
    a, b = a.double(), b.double()
    assert torch.isfinite(a).all(), name
    assert (a - b).norm() <= 4 * 2 ** -9 * b.norm() + 1e-5 * b.numel() ** 0.5, name


def rows_close(a, b, name):
    a, b = a.double(), b.double()
    if name == "lse":
        assert (a - b).abs().max() <= 2 * 2 ** -9 + 1e-5, name
        return
    bound = (16 if name == "O" else 2) * 2 ** -9 * b.norm(dim=-1) + 1e-5 * b.shape[-1] ** 0.5
    assert ((a - b).norm(dim=-1) <= bound).all(), name


# left: tiles of the forward's last round, of 256 query rows but for the last case, whose blocks have 384
@pytest.mark.parametrize("nq,nk,H,left", [
    ([1], [1], 1, 1), ([300, 5, 70], [300, 5, 700], 1, 4),        # 8 pieces each, most of them empty
    ([200, 257, 0, 600], [500, 0, 64, 449], 3, 18),               # sides without rows
    ([256] * 32 + [1], [90] * 33, 1, 33),                         # 7 pieces
    ([256] * 64, [130] * 64, 2, 128), ([256] * 43, [130] * 43, 3, 129),   # two pieces; none
    ([100] * 257, None, 1, 0),                                    # a round (dK/dV: and one tile)
    ([100] * 255 + [300], None, 1, 1), ([100] * 255, None, 1, 255),   # a round and one tile; a tile less than a round
    ([3000, 2500, 100], None, 12, 192),                           # none (dK/dV, 192 keys: a round, and two pieces)
])
def test_split_against_whole_tiles(nq, nk, H, left):
    nk = nk or nq
    if len(nq) > 256:
        nq, nk = nq[:255] + [sum(nq[255:])], nk[:255] + [sum(nk[255:])]
    rows = 384 if len(nq) == 3 and nq[0] == 3000 else 256
    assert sum(-(-n // rows) for n in nq) * H % 256 == left
    g = torch.Generator().manual_seed(len(nq) + H)
    Nq, Nk, G = sum(nq), sum(nk), len(nq)
    q, d = (torch.randn((H, Nq, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    k, v = (torch.randn((H, Nk, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    cq, ck = (torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int32)).cuda() for n in (nq, nk))
    s = 128 ** -0.5
    lib, stream = mg.load(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    mg.set_small_group_rows(0)   # the kernels with long blocks, whatever the mean size
    try:
        out = {}
        for op, name in ((mg.OP_VARLEN_ATTN_FWD, "fwd"), (mg.OP_VARLEN_ATTN_BWD, "bwd")):
            need = mg.workspace_bytes(op, Nq, H, 128, G, 0, mg.MOGA_BF16)
            pref = lib.moga_workspace_preferred_bytes(op, Nq, Nk, H, 128, G, 0, mg.MOGA_BF16)
            assert pref > need and mg.attn_blocks(op, Nq, Nk, H, G, pref)[:2] == (rows, True)
            for size in (need, pref):
                ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN wherever nothing is written
                if name == "fwd":
                    oh, lse = torch.empty_like(q), torch.empty((H, Nq), device="cuda")
                    st = lib.moga_varlen_attn_fwd(p(q), p(k), p(v), mg.MOGA_BF16, Nq, Nk, H, 128, p(cq), p(ck), G, s, p(oh), p(lse),
                                                  p(ws), size, stream)
                    out[size == pref] = [oh, lse]
                else:
                    o, l = out[False][:2]
                    gr = [torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)]
                    st = lib.moga_varlen_attn_bwd(p(d), p(q), p(k), p(v), p(o), p(l), mg.MOGA_BF16, Nq, Nk, H, 128, p(cq), p(ck), G, s,
                                                  *(p(t) for t in gr), p(ws), size, stream)
                    out[size == pref] += gr
                assert st == 0
        torch.cuda.synchronize()
    finally:
        mg.set_small_group_rows(-1)
    none = out[False][1] == -torch.inf   # queries without keys
    assert torch.equal(out[True][1] == -torch.inf, none)
    for t in out.values():
        t[1] = t[1].masked_fill(none, 0.0)
    for a, b, name in zip(out[True], out[False], ("O", "lse", "dQ", "dK", "dV")):
        close(a, b, name)
        rows_close(a, b, name)
    if none.any():
        assert (out[True][0][none] == 0).all() and (out[True][2][none] == 0).all()


def test_call_on_another_stream_takes_no_workspace_of_this_one():
    g = torch.Generator().manual_seed(3)
    q, k, v = (torch.randn((12, 8000, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    cu = torch.tensor([0, 4100, 8000], dtype=torch.int32, device="cuda")
    assert mg.load().moga_workspace_preferred_bytes(mg.OP_ATTN_FWD, 8000, 8000, 12, 128, 2, 0, mg.MOGA_BF16) > 0
    mg.set_small_group_rows(0)
    try:
        ref, _ = mg.moga_group_attn_fwd(q, k, v, cu, 128 ** -0.5)   # split
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        got, lse = mg.moga_group_attn_fwd(q, k, v, cu, 128 ** -0.5, stream=side)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before + 2   # the two outputs
        torch.cuda.current_stream().wait_stream(side)
        close(got, ref, "O")
        torch.cuda.synchronize()
    finally:
        mg.set_small_group_rows(-1)


# groups that take blocks of 256 and of 384 query rows
@pytest.mark.parametrize("nq,rows", [([300, 900], 256), ([2083, 4412], 384)])
@pytest.mark.parametrize("what", ["nan query", "nan key", "inf score", "all scores -inf", "inf value"])
def test_split_keeps_nan_and_infinities(what, nq, rows):
    """One row of Q, K or V that is not finite: NaN and infinities come out at the same places as from whole tiles."""
    print(what, nq, flush=True)
    H, s = 2, 128 ** -0.5
    N = sum(nq)
    g = torch.Generator().manual_seed(7)
    q, k, v = (torch.randn((H, N, 128), generator=g) for _ in range(3))
    if what == "nan query":
        q[0, 40] = torch.nan
    elif what == "nan key":
        k[1, nq[0] + 10] = torch.nan
    elif what == "inf score":
        k[0, 17] = 3e38
        q[0, 5] = 1.0
    elif what == "all scores -inf":
        k[0, :nq[0]] = -k[0, :nq[0]].abs()
        q[0, 5] = 3e38
    else:
        v[1, nq[0] + 100, 3] = torch.inf
    q, k, v = (t.to(torch.bfloat16).cuda() for t in (q, k, v))
    cu = torch.tensor([0, nq[0], N], dtype=torch.int32, device="cuda")
    lib, stream = mg.load(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    mg.set_small_group_rows(0)
    try:
        out = []
        assert mg.attn_blocks(mg.OP_VARLEN_ATTN_FWD, N, N, H, 2, 1 << 30)[:2] == (rows, True)
        for size in (mg.workspace_bytes(mg.OP_VARLEN_ATTN_FWD, N, H, 128, 2, 0, mg.MOGA_BF16),
                     lib.moga_workspace_preferred_bytes(mg.OP_VARLEN_ATTN_FWD, N, N, H, 128, 2, 0, mg.MOGA_BF16)):
            ws, oh, lse = torch.empty(size, dtype=torch.uint8, device="cuda"), torch.empty_like(q), torch.empty((H, N), device="cuda")
            assert lib.moga_varlen_attn_fwd(p(q), p(k), p(v), mg.MOGA_BF16, N, N, H, 128, p(cu), p(cu), 2, s, p(oh), p(lse), p(ws), size,
                                            stream) == 0
            out.append((oh, lse))
        torch.cuda.synchronize()
    finally:
        mg.set_small_group_rows(-1)
    (o0, l0), (o1, l1) = out
    assert not (torch.isfinite(o0).all() and torch.isfinite(l0).all())
    for a, b in ((o0, o1), (l0, l1)):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
        assert torch.equal(a[torch.isinf(a)], b[torch.isinf(b)])
        fin = torch.isfinite(a)
        close(b[fin], a[fin], what)


def test_forward_without_ws_leaves_the_workspace_alone():
    """moga_group_attn_fwd needs no workspace: what a caller passes all the same may be in use on other streams."""
    N, H, s = 6000, 4, 128 ** -0.5
    g = torch.Generator().manual_seed(1)
    q, k, v = (torch.randn((H, N, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    lib, stream = mg.load(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    mg.set_small_group_rows(0)
    try:
        size = lib.moga_workspace_preferred_bytes(mg.OP_ATTN_FWD, N, N, H, 128, 1, 0, mg.MOGA_BF16)
        used = []
        for fn in (lib.moga_group_attn_fwd, lib.moga_group_attn_fwd_ws):
            ws, oh, lse = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda"), torch.empty_like(q), torch.empty((H, N), device="cuda")
            assert fn(p(q), p(k), p(v), mg.MOGA_BF16, N, H, 128, p(cu), 1, s, p(oh), p(lse), p(ws), size, stream) == 0
            used.append(bool((ws != 0x5A).any()))
        torch.cuda.synchronize()
    finally:
        mg.set_small_group_rows(-1)
    assert used == [False, True]


def varlen_results(nq, nk, H, bytes_of, o_lse=None, seed=0):
    """O, lse, dQ, dK, dV of the varlen calls with bytes_of(needed, preferred) bytes of workspace, of which the bytes past them stay as they
    are, and the blocks that they took.  The backward takes o_lse if given (the bounds of rows_close want P and dS alike on both sides)."""
    g = torch.Generator().manual_seed(len(nq) + H + seed)
    Nq, Nk, G = sum(nq), sum(nk), len(nq)
    q, d = (torch.randn((H, Nq, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    k, v = (torch.randn((H, Nk, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    cq, ck = (torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int32)).cuda() for n in (nq, nk))
    s, lib, stream = 128 ** -0.5, mg.load(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    took, out = [], [torch.empty_like(q), torch.empty((H, Nq), device="cuda"), torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)]
    for op in (mg.OP_VARLEN_ATTN_FWD, mg.OP_VARLEN_ATTN_BWD):
        need = mg.workspace_bytes(op, Nq, H, 128, G, 0, mg.MOGA_BF16)
        size = bytes_of(need, lib.moga_workspace_preferred_bytes(op, Nq, Nk, H, 128, G, 0, mg.MOGA_BF16))
        ws = torch.full((size + 4096,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN wherever nothing is written
        if op == mg.OP_VARLEN_ATTN_FWD:
            st = lib.moga_varlen_attn_fwd(p(q), p(k), p(v), mg.MOGA_BF16, Nq, Nk, H, 128, p(cq), p(ck), G, s, p(out[0]), p(out[1]), p(ws), size,
                                          stream)
        else:
            st = lib.moga_varlen_attn_bwd(p(d), p(q), p(k), p(v), *(p(t) for t in o_lse or out[:2]), mg.MOGA_BF16, Nq, Nk, H, 128, p(cq), p(ck), G, s,
                                          *(p(t) for t in out[2:]), p(ws), size, stream)
        assert st == 0 and (ws[size:] == 0xFF).all()
        took.append(mg.attn_blocks(op, Nq, Nk, H, G, size))
    torch.cuda.synchronize()
    return out, took


@pytest.fixture
def large_kernels():
    mg.set_small_group_rows(0)   # the kernels with long blocks, whatever the mean size
    yield
    mg.set_small_group_rows(-1)


def test_room_for_short_pieces(large_kernels):
    """34 MB past what a call needs: pieces of 256 rows where it would take 384 with more."""
    n = [1700, 1600, 2]
    print(n, flush=True)
    short = 256 + 256 * 256 * 130 * 4
    whole, _ = varlen_results(n, n, 6, lambda need, pref: need)
    less, took = varlen_results(n, n, 6, lambda need, pref: need + short, whole[:2])
    assert took == [(256, True, 0, False), (256, True, 128, True)]
    for a, b, name in zip(less, whole, ("O", "lse", "dQ", "dK", "dV")):
        rows_close(a, b, name)


# Blocks of 384 query rows (forward, dQ) and of `keys` keys; left: their tiles in the last round
@pytest.mark.parametrize("n,H,left,keys,keys_left", [
    ([2083, 4412], 2, 36, 192, 68), ([3803], 6, 60, 192, 120),                      # 7 and 4 pieces; 3 and 2
    ([6144, 6144], 4, 128, 192, 0), ([384] * 43, 3, 129, 128, 131),                 # two pieces; none
    ([384] * 64 + [1], 4, 4, 192, 4),                                               # a round (dK/dV: two) and a few tiles
    ([700] * 15, 12, 104, 192, 208), ([3000, 2500, 100], 12, 192, 192, 116),        # a round and more
])
def test_split_of_long_blocks_against_whole_tiles(large_kernels, n, H, left, keys, keys_left):
    print(n, H, flush=True)
    whole, none = varlen_results(n, n, H, lambda need, pref: need)
    pieces, took = varlen_results(n, n, H, lambda need, pref: pref, whole[:2])
    assert not any(b[1] or b[3] for b in none) and took == [(384, True, 0, False), (384, True, keys, True)]
    assert sum(-(-i // 384) for i in n) * H % 256 == left and sum(-(-i // keys) for i in n) * H % 256 == keys_left
    for a, b, name in zip(pieces, whole, ("O", "lse", "dQ", "dK", "dV")):
        close(a, b, name)
        rows_close(a, b, name)
