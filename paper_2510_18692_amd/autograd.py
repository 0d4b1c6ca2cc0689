"""torch.autograd wrappers around the C-ABI calls (argument marshalling only).

    o, lb = moga_attention(x, w, q, k, v, scale, balance_alpha=0.1)

`o` is the output of Alg. 1 with the gate of Eq. 5, `lb` the group balancing loss of Eqs. 6-8 (or
None).  Gradients flow to q, k, v and to the router weight w (through the gate, and through the
balancing loss when it is used); the assignment itself is a constant of differentiation.  No
gradient is returned for the router input x unless `grad_x=True` (the optional dX of the router
backward).  Everything runs in the HIP library; the autograd function itself is native
(csrc/torch_binding.cpp), so that the backward pass does not enter the interpreter.
"""
from __future__ import annotations

from . import binding as mg


def moga_attention(x, w, q, k, v, softmax_scale, balance_alpha=None, grad_x=False):
    """x [N, d_model], w [M, d_model] fp32, q/k/v [N, H, D] -> (o [N, H, D], balancing loss or None, group [N])."""
    o, loss, group = mg._nat.attention(x, w, q, k, v, softmax_scale, balance_alpha, grad_x)
    return o, (loss if balance_alpha is not None else None), group
