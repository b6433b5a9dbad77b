"""The autograd wrapper returns the library's forward and routes gradients through flare_backward:
checked against the fp64 oracle's forward and backward on the same seeded inputs."""
import numpy as np
import pytest

from paper_2508_12594_amd import synth
from paper_2508_12594_amd.autograd import flare_mixer
from tests._util import slice_relerr, to_device, to_host, tol_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,over,layout,y_f32", [(1, dict(N=600), "bhnd", False), (2, dict(B=2, N=1500), "bhnd", False),
                                                   (4, dict(N=1200, dtype="f16"), "bnhd", False),
                                                   (2, dict(B=2, N=1500, d=8), "bnhd", True)])
def test_autograd_matches_oracle(oracle, cfg, over, layout, y_f32):
    import torch
    print("[case] autograd cfg%d %s %s" % (cfg, over, layout), flush=True)
    inp = synth.make_inputs(cfg, with_dy=True, **over)
    scale, tol = inp["scale"], tol_for(inp)
    dev = to_device(inp)
    conv = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
    back = (lambda t: t.permute(0, 2, 1, 3)) if layout == "bnhd" else (lambda t: t)
    q = dev["q"].clone().requires_grad_(True)
    k = conv(dev["k"]).clone().requires_grad_(True)
    v = conv(dev["v"]).clone().requires_grad_(True)
    y = flare_mixer(q, k, v, scale, layout=layout, y_f32=y_f32)
    assert y.dtype == (torch.float32 if y_f32 else k.dtype)
    y.backward(conv(dev["dy"]).to(y.dtype))
    torch.cuda.synchronize()
    y_ref, _, _ = oracle.forward(inp["q"], inp["k"], inp["v"], scale)
    dq_ref, dk_ref, dv_ref = oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)
    assert q.grad.dtype == q.dtype and k.grad.shape == k.shape
    errs = dict(y=slice_relerr(to_host(back(y)), y_ref), dq=slice_relerr(to_host(q.grad), dq_ref),
                dk=slice_relerr(to_host(back(k.grad)), dk_ref), dv=slice_relerr(to_host(back(v.grad)), dv_ref))
    print("[case]    " + "  ".join("%s %.2e" % kv for kv in errs.items()), flush=True)
    # dq_lat is cast to q's dtype for autograd: one more rounding of a 16-bit type
    assert max(errs.values()) <= tol


def test_autograd_hooks_and_refusals():
    """Saved tensors pass through the caller's hooks, a second backward without retain_graph and an in-place change of
    the output are errors, a forward-mode tangent is refused, and threads may call at the same time."""
    import threading

    import torch
    import torch.autograd.forward_ad as fwad
    print("[case] autograd hooks", flush=True)
    inp = synth.make_inputs(2, B=1, H=2, N=300, M=32, d=16, dtype="bf16", with_dy=True)
    dev = to_device(inp)
    scale = inp["scale"]

    def step(packed=None):
        q, k, v = (dev[n].clone().requires_grad_(True) for n in ("q", "k", "v"))
        pack = (lambda t: packed.append(t) or t) if packed is not None else (lambda t: t)
        with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t.clone()):
            y = flare_mixer(q, k, v, scale)
        return y, torch.autograd.grad(y, (q, k, v), dev["dy"])

    packed = []
    y, grads = step(packed)
    assert len(packed) == 5
    results = [None] * 4

    def work(i):
        results[i] = step()
        torch.cuda.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    for y2, grads2 in results:
        assert torch.equal(y, y2) and all(torch.equal(a, b) for a, b in zip(grads, grads2))

    q = dev["q"].clone().requires_grad_(True)
    y = flare_mixer(q, dev["k"], dev["v"], scale)
    torch.autograd.grad(y, q, dev["dy"], retain_graph=True)
    torch.autograd.grad(y, q, dev["dy"])
    with pytest.raises(RuntimeError):
        torch.autograd.grad(y, q, dev["dy"])
    y = flare_mixer(q, dev["k"], dev["v"], scale)
    y.mul_(2.0)
    with pytest.raises(RuntimeError):
        torch.autograd.grad(y, q, dev["dy"])
    with fwad.dual_level():
        dual = fwad.make_dual(dev["q"], torch.ones_like(dev["q"]))
        with pytest.raises(RuntimeError):
            flare_mixer(dual, dev["k"], dev["v"], scale)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda t: flare_mixer(dev["q"], t, t, scale))(torch.stack([dev["k"], dev["k"]]))


@pytest.mark.parametrize("dtype,shared,layout,y_f32", [("f32", False, "bhnd", False), ("bf16", True, "bnhd", False),
                                                       ("f16", False, "bhnd", True)])
def test_unpacked_tensors_are_held_against_the_forward(dtype, shared, layout, y_f32):
    """A saved-tensor hook that hands back another type, shape, order or device for any one of the saved tensors is an
    error before anything is launched; handing back equal copies is not."""
    import torch

    from paper_2508_12594_amd.binding import FlareError
    print("[case] unpacked tensors %s shared=%s %s y_f32=%s" % (dtype, shared, layout, y_f32), flush=True)
    inp = synth.make_inputs(2, B=1, H=2, N=300, M=32, d=16, dtype=dtype, with_dy=True)
    dev = to_device(inp)
    order = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
    k, v, dy = (order(dev[n]) for n in ("k", "v", "dy"))
    q = (dev["q"][0].contiguous() if shared else dev["q"]).requires_grad_(True)

    def gradient(which, change):
        count = [0]

        def unpack(t):
            count[0] += 1
            return change(t) if count[0] - 1 == which else t.clone()

        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, unpack):
            y = flare_mixer(q, k, v, inp["scale"], layout=layout, y_f32=y_f32)
        dq, = torch.autograd.grad(y, q, dy.float() if y_f32 else dy)
        assert count[0] == 5
        return dq

    y = flare_mixer(q, k, v, inp["scale"], layout=layout, y_f32=y_f32)
    dq_ref, = torch.autograd.grad(y, q, dy.float() if y_f32 else dy)
    assert torch.equal(gradient(-1, None), dq_ref)
    changes = [lambda t: t.to(torch.float64), lambda t: t.flatten()[:-64].clone(),
               lambda t: t.unsqueeze(0), lambda t: torch.stack([t, t], -1)[..., 0], lambda t: t.cpu()]
    for which in range(5):
        for change in changes:
            with pytest.raises(FlareError):
                gradient(which, change)
    for which in range(4):                      # 16 bits, or single precision, that was not undone
        with pytest.raises(FlareError):
            gradient(which, lambda t: t.half() if t.dtype == torch.float32 else t.float())
    assert torch.equal(gradient(-1, None), dq_ref)


@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("dtype,layout,y_f32", [("f32", "bhnd", False), ("bf16", "bnhd", False), ("bf16", "bhnd", True)])
def test_traced_mixer_is_an_operation(dtype, layout, y_f32, grad):
    """torch.jit.trace records the mixer, under no_grad too: the traced function gives other inputs (and another number of
    tokens) their own output and gradients, the bits of a direct call."""
    import torch
    print("[case] jit.trace %s %s y_f32=%s grad=%s" % (dtype, layout, y_f32, grad), flush=True)

    def draw(N, seed):
        inp = synth.make_inputs(2, B=1, H=2, N=N, M=32, d=16, dtype=dtype, with_dy=True, seed=seed)
        dev = to_device(inp)
        order = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
        return inp["scale"], [dev["q"]] + [order(dev[n]) for n in ("k", "v", "dy")]

    scale, (q, k, v, _) = draw(300, 1)

    def layer(a, b, c):
        return flare_mixer(a, b, c, scale, layout=layout, y_f32=y_f32) * 2.0

    with torch.set_grad_enabled(grad):
        traced = torch.jit.trace(layer, (q, k, v))
    for N, seed in ((300, 1), (300, 2), (77, 3)):
        _, (q, k, v, dy) = draw(N, seed)
        dy = dy.float() if y_f32 else dy
        for t in (q, k, v):
            t.requires_grad_(True)
        y, y_ref = traced(q, k, v), layer(q, k, v)
        assert torch.equal(y, y_ref)
        for a, b in zip(torch.autograd.grad(y, (q, k, v), dy), torch.autograd.grad(y_ref, (q, k, v), dy)):
            assert torch.equal(a, b)
        with torch.no_grad():
            assert torch.equal(traced(q, k, v), y_ref)


def test_nothing_came_back_to_the_output():
    """A consumer of y whose backward returns no gradient: the gradients are zeros, not missing."""
    import torch
    print("[case] undefined gradient", flush=True)

    class Detour(torch.autograd.Function):
        @staticmethod
        def forward(ctx, x):
            return x.clone()

        @staticmethod
        def backward(ctx, g):
            return None

    inp = synth.make_inputs(2, B=1, H=2, N=300, M=32, d=16, dtype="bf16")
    q, k, v = (t.requires_grad_(True) for t in to_device(inp, ("q", "k", "v")).values())
    for y_f32 in (False, True):
        y = Detour.apply(flare_mixer(q, k, v, inp["scale"], y_f32=y_f32))
        for t, g in zip((q, k, v), torch.autograd.grad(y, (q, k, v), torch.ones_like(y))):
            assert g.dtype == t.dtype and g.shape == t.shape and not g.any()
