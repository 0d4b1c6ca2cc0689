"""What users of the library have it do, as measurable cases.

A case is one pass of Mixture-of-Groups attention through the public entry points of
`paper_2510_18692_amd`: inference (`moga_forward`), a training step (`moga_forward` +
`moga_backward`), a training step through autograd with the balancing loss
(`moga_attention`), a training step that never materialises the permuted tensors
(`moga_fused_attn_fwd` / `_bwd`), or a training step of the three-branch block
(`visual_forward` + `visual_backward`).  Token counts, widths and group counts are those of
`workloads.py`, of the tests and of `bench.py`: latent frames of 30 x 52 = 1,560 tokens, the
1536/12 and 5120/40 (width / heads) backbones, 1 to 32 groups, contexts from one frame to
580,320 tokens.
"""
from __future__ import annotations

import math

import torch

from paper_2510_18692_amd import binding as mg
from paper_2510_18692_amd import workloads as wl
from paper_2510_18692_amd.autograd import moga_attention

FRAME = (30, 52)   # latent frame of 480p video, rows x columns


def listed():
    """The cases, smallest first.  `hidden`: how the router input is distributed (see workloads.py)."""
    tiny = dict(N=4096, H=2, D=64, d_model=128, M=8, dtype="f32", hidden="iid")
    wide = dict(H=40, D=128, d_model=5120, dtype="bf16", hidden="mixture")
    clip = dict(H=12, D=128, d_model=1536, dtype="bf16", hidden="iid")
    return [
        # full-precision inference and training at the size unit tests and gradient checks of a model use
        dict(name="tiny_f32_infer", kind="infer", **tiny),
        dict(name="tiny_f32_train", kind="train", **tiny),
        # the smallest bf16 call: one latent frame (an image), autograd step with the balancing loss
        dict(name="one_frame_autograd", kind="autograd", N=1560, H=4, D=128, d_model=512, M=8, dtype="bf16",
             hidden="iid", grad_x=False),
        # a short context of no round size: fine-tuning on mixed-length clips, twenty groups
        dict(name="ragged_train", kind="train", **{**clip, "N": 10007, "M": 20}),
        # 21 latent frames on the small backbone: one denoising step of inference
        dict(name="clip_infer", kind="infer", **{**clip, "N": 32760, "M": 8}),
        # 40 latent frames (ten seconds), five groups, gradient of the hidden state included
        dict(name="ten_seconds_autograd", kind="autograd", **{**clip, "N": 62400, "M": 5}, grad_x=True),
        # the three-branch block on a 21-frame clip: 2 x 2 spatial windows, three shots
        dict(name="clip_block", kind="block", **{**clip, "N": 32760, "M": 5}, shots=3, wh=15, ww=26),
        # 64 frames on the large backbone, group sizes that span 46x, two nearly empty groups
        dict(name="unbalanced_train", kind="train", N=99840, M=16, weights="zipf", zipf_s=1.45, absent=2, align=5.0, **wide),
        # the same context without permuted tensors in memory, Zipf(1.1) groups
        dict(name="fused_train", kind="fused", N=99840, M=16, weights="zipf", **wide),
        # the three-branch block on 64 frames: 4 x 4 spatial windows, four shots
        dict(name="long_block", kind="block", N=99840, M=16, shots=4, wh=8, ww=13, **wide),
        # paper-scale context, one inference pass and one training step
        dict(name="paper_scale_infer", kind="infer", N=580320, M=32, noise_var=0.5, **wide),
        dict(name="paper_scale_train", kind="train", N=580320, M=32, noise_var=0.5, **wide),
    ]


def draw(rng):
    """One more case: any kind, context length spread over its logarithm, odd lengths among them."""
    kind = rng.choice(["infer", "train", "autograd", "fused", "block"])
    if kind in ("infer", "train") and rng.random() < 0.35:   # full precision: small contexts
        D = rng.choice([64, 64, 128])
        return dict(kind=kind, N=int(math.exp(rng.uniform(math.log(256), math.log(8192)))), H=rng.randint(1, 4), D=D,
                    d_model=rng.choice([64, 96, 128, 200, 256]), M=rng.choice([2, 5, 8, 16, 20]), dtype="f32",
                    hidden="iid")
    wide = rng.random() < 0.4
    case = dict(kind=kind, H=40 if wide else rng.choice([3, 4, 12, 12, 16]), D=128,
                d_model=5120 if wide else rng.choice([512, 1536, 1536, 1536]), dtype="bf16")
    case["M"] = rng.choice([2, 4, 5, 8, 10, 16, 20, 32])
    case["hidden"] = rng.choice(["iid", "mixture", "mixture"])
    if case["hidden"] == "mixture" and rng.random() < 0.5:
        case.update(weights="zipf", zipf_s=rng.choice([1.1, 1.45]))
    if kind == "block":
        frames = int(math.exp(rng.uniform(math.log(2), math.log(64))))
        wh, ww = rng.choice([(15, 26), (8, 13), (7, 13), (10, 18)])
        case.update(N=frames * FRAME[0] * FRAME[1], shots=rng.randint(1, min(4, frames)), wh=wh, ww=ww)
    else:
        case["N"] = int(math.exp(rng.uniform(math.log(700), math.log(200000))))
    if kind == "autograd":
        case["grad_x"] = rng.random() < 0.5
    # no more work than the largest listed case
    most = max(work(c)["flops"] for c in listed())
    while work(case)["flops"] > 0.25 * most:
        case["N"] //= 2
        if kind == "block":
            case["N"] = max(2 * FRAME[0] * FRAME[1], case["N"] // (FRAME[0] * FRAME[1]) * FRAME[0] * FRAME[1])
            case["shots"] = 1
    return case


def _workload(case, seed=0):
    keys = ("N", "H", "D", "d_model", "M", "dtype", "hidden", "weights", "zipf_s", "absent", "align", "noise_var")
    return wl.Workload(name=case["kind"], backward=case["kind"] != "infer", seed=seed,
                       **{k: case[k] for k in keys if k in case})


def prepare(case, seed):
    """Inputs on the GPU and, for the block, the static index lists: what a program holds before the call."""
    w = _workload(case, seed)
    inp = wl.make_inputs(w, "cuda")
    st = {"kind": case["kind"], "scale": w.scale, "M": w.M}
    st.update({k.lower() if k != "dO" else k: inp[k] for k in ("X", "W", "Q", "K", "V", "dO") if k in inp})
    if case["kind"] == "autograd":
        st["grad_x"] = case["grad_x"]
        st["one"] = torch.ones((), device="cuda")
        st["wrt"] = [st["w"], st["q"], st["k"], st["v"]] + ([st["x"]] if case["grad_x"] else [])
        for t in st["wrt"]:
            t.requires_grad_(True)
    elif case["kind"] == "block":
        T = case["N"] // (FRAME[0] * FRAME[1])
        st["grid"] = (T, *FRAME)
        shot_of_frame = [t * case["shots"] // T for t in range(T)]
        st["static"] = mg.moga_stga_build_index(T, *FRAME, case["wh"], case["ww"], T, shot_of_frame)
    return st


def run(s):
    """One pass; outputs in token order."""
    kind = s["kind"]
    if kind == "infer":
        f = mg.moga_forward(s["x"], s["w"], s["q"], s["k"], s["v"], s["scale"], want_probs=False)
        return {"o": f["o"], "group": f["group"]}
    if kind == "train":
        f = mg.moga_forward(s["x"], s["w"], s["q"], s["k"], s["v"], s["scale"])
        b = mg.moga_backward(f, s["x"], s["w"], s["dO"], s["scale"])
        return {"o": f["o"], **{k: b[k] for k in ("d_q", "d_k", "d_v", "d_w")}}
    if kind == "autograd":
        o, loss, _ = moga_attention(s["x"], s["w"], s["q"], s["k"], s["v"], s["scale"], balance_alpha=0.1,
                                    grad_x=s["grad_x"])
        return {"o": o, "loss": loss, "grads": list(torch.autograd.grad([o, loss], s["wrt"], [s["dO"], s["one"]]))}
    if kind == "fused":
        group, gate, probs, _ = mg.moga_route(s["x"], s["w"])
        pm = mg.moga_permute(group, s["M"])
        o, lse = mg.moga_fused_attn_fwd(s["q"], s["k"], s["v"], pm["perm"], gate, pm["cu_seqlens"], s["scale"])
        d_q, d_k, d_v, d_gate = mg.moga_fused_attn_bwd(s["dO"], s["q"], s["k"], s["v"], o, lse, pm["perm"],
                                                       pm["inv_perm"], gate, pm["cu_seqlens"], s["scale"])
        d_w, _ = mg.moga_route_bwd(s["x"], s["w"], probs, group, gate, d_gate)
        return {"o": o, "d_q": d_q, "d_k": d_k, "d_v": d_v, "d_w": d_w}
    f = mg.visual_forward(s["x"], s["w"], s["q"], s["k"], s["v"], s["scale"], s["grid"], s["static"])
    b = mg.visual_backward(f, s["x"], s["w"], s["dO"], s["scale"])
    return {"o": f["o"], **{k: b[k] for k in ("d_q", "d_k", "d_v", "d_w")}}


def _static_pairs(case):
    """Query-key pairs of the spatial-temporal and the per-frame groups of a block case."""
    fh, fw = FRAME
    T = case["N"] // (fh * fw)
    sides = [[min(s, n - i) for i in range(0, n, s)] for n, s in ((fh, case["wh"]), (fw, case["ww"]))]
    windows = [a * b for a in sides[0] for b in sides[1]]
    length = [0] * case["shots"]
    for t in range(T):
        length[t * case["shots"] // T] += 1
    frames = sum(n * (n + (i > 0) + (i + 1 < len(length))) for i, n in enumerate(length))
    return frames * sum(a * a for a in windows) + T * (fh * fw) ** 2


def work(case):
    """Attention inside the groups (expected sizes) and the two router products; every tensor once."""
    N, H, D, d, M = (case[k] for k in ("N", "H", "D", "d_model", "M"))
    es = 4 if case["dtype"] == "f32" else 2
    train = case["kind"] != "infer"
    p = [1.0] * M
    if case.get("weights") == "zipf":
        p = [(k + 1) ** -case.get("zipf_s", 1.1) if k < M - case.get("absent", 0) else 0.0 for k in range(M)]
    pairs = N * N * sum(v * v for v in p) / sum(p) ** 2
    if case["kind"] == "block":
        pairs += _static_pairs(case)
    grad_x = case.get("grad_x", False)
    flops = (14 if train else 4) * H * D * pairs + 2.0 * N * d * M * (1 + train + grad_x)
    rows = N * H * D * es
    size = N * d * es + M * d * 4 + 4 * rows
    if train:
        size += 4 * rows + M * d * 4 + (N * d * es if grad_x else 0)
    return {"bytes": float(size), "flops": float(flops)}


def tolerance(case):
    """About four times what the path differs by from a float64 evaluation of the same inputs.

    Measured with torch in float64 at 1,560 to 8,000 tokens over every kind: fp32 outputs and gradients 0.6e-6 to
    1.2e-6 in the 2-norm and up to 0.9e-5 at one element; bf16 2.1e-3 to 3.4e-3 in the 2-norm (bf16 P, dS and
    outputs) and up to 0.055 at one element.  No token changed its group; a tie may.
    """
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5, "differ": 1e-4}
    return {"rel": 1.3e-2, "max": 0.2, "differ": 1e-4}
