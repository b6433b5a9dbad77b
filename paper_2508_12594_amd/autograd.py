"""torch.autograd wrapper around the binding: `flare_mixer(q_lat, k, v, scale)` is differentiable.

Nothing is computed here: the forward calls flare_forward (keeping z, lse_enc, lse_dec and y for the
backward), the backward calls flare_backward_cast (dq_lat in q_lat's dtype, which autograd requires of a
gradient).  The autograd node is native (csrc/torch_binding.cpp, MixerBackward).  This is how the paper's layer
would use the operator in place of its two attention calls (listing in Section 3.1).
"""
from . import binding


def flare_mixer(q_lat, k, v, scale, layout="bhnd", y_f32=False):
    """y = FLARE(q_lat, k, v): q_lat [H,M,d] (or [M,d]: shared latents), k, v [B,H,N,d] ('bhnd') or
    [B,N,H,d] ('bnhd'); returns y in k's shape and dtype.  Differentiable in q_lat, k and v.

    y_f32 (16-bit inputs, at most 2048 latents): y comes back in fp32 and the backward reads it instead of
    recomputing the token statistics, which pays at d < 16 (flare_shape.y_f32)."""
    return binding._native().mixer(q_lat, k, v, float(scale), binding._layout(layout), bool(y_f32))
