"""GPU parity for the [B,N,H,d] layout of the token tensors (k, v, y, dy, dk, dv as the block's
linear projections leave them, before any head transpose).

Two checks per case: against the fp64 oracle on the same seeded inputs (the oracle always takes
[B,H,N,d]; the test transposes, which is data movement only), and bit for bit against the
library's own [B,H,N,d] run, since the arithmetic does not depend on where a row lives.
"""
import sys

import numpy as np
import pytest

from paper_2508_12594_amd import binding, synth
from tests._util import slice_relerr, to_device, to_host, tol_for

pytestmark = pytest.mark.gpu


def _say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


def _bnhd(t):
    return t.permute(0, 2, 1, 3).contiguous()


CASES = [
    (1, dict(N=777, B=2)),          # fp32 storage
    (1, dict(N=300, M=40, d=4)),    # smallest head dimension, ragged M
    (2, dict(B=2, N=2050)),         # matrix-core path, d=16, M=64
    (3, dict(B=2, N=1500)),         # d=32, M=128
    (4, dict(N=5003)),              # d=16, M=256
    (5, dict(N=2001)),              # d=32, M=256
    (4, dict(N=33, H=3)),           # odd head count, two tiles
    (2, dict(B=1, N=1200, d=8)),    # matrix-core path with the head dimension padded to 16
    (4, dict(N=700, d=4, H=4)),
    (2, dict(B=1, N=900, M=512)),                # latent chunks on the matrix-core path
    (1, dict(N=400, M=72, dtype="f16")),         # fp16 storage, 8 padding latents
    (4, dict(N=1100, dtype="f16")),              # fp16 storage, matrix-core path
    (5, dict(N=700, dtype="f16")),
]


@pytest.mark.parametrize("saved", [True, False])
@pytest.mark.parametrize("cfg,over", CASES)
def test_token_major_layout(oracle, cfg, over, saved):
    import torch
    _say("layout bnhd cfg%d %s saved=%s" % (cfg, over, saved))
    inp = synth.make_inputs(cfg, with_dy=True, **over)
    scale, tol = inp["scale"], tol_for(inp)
    dev = to_device(inp)
    B, H, N, _ = dev["k"].shape

    def run(layout):
        conv = _bnhd if layout == "bnhd" else (lambda t: t)
        k, v, dy = conv(dev["k"]), conv(dev["v"]), conv(dev["dy"])
        lse_dec = torch.empty((B, H, N), dtype=torch.float32, device="cuda") if saved else None
        y, z, lse = binding.forward(dev["q"], k, v, scale, lse_dec=lse_dec, layout=layout)
        dq, dk, dv = binding.backward(dev["q"], k, v, dy, z, lse, scale, y=y if saved else None,
                                      lse_dec=lse_dec, layout=layout)
        torch.cuda.synchronize()
        back = (lambda t: t.permute(0, 2, 1, 3)) if layout == "bnhd" else (lambda t: t)
        assert y.shape == k.shape and dk.shape == k.shape and dv.shape == k.shape
        return dict(y=back(y), z=z, lse=lse, dq=dq, dk=back(dk), dv=back(dv),
                    lse_dec=lse_dec if saved else torch.zeros(1))

    got = run("bnhd")
    same = run("bhnd")
    for name in got:
        assert torch.equal(got[name], same[name]), "%s differs between the two layouts" % name

    y_ref, z_ref, lse_ref = oracle.forward(inp["q"], inp["k"], inp["v"], scale)
    dq_ref, dk_ref, dv_ref = oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)
    errs = dict(y=slice_relerr(to_host(got["y"]), y_ref), z=slice_relerr(to_host(got["z"]), z_ref),
                dq=slice_relerr(to_host(got["dq"]), dq_ref), dk=slice_relerr(to_host(got["dk"]), dk_ref),
                dv=slice_relerr(to_host(got["dv"]), dv_ref))
    _say("   " + "  ".join("%s %.3e" % kv for kv in errs.items()) + "  (tol %.0e)" % tol)
    assert max(errs.values()) <= tol
    assert float(np.max(np.abs(to_host(got["lse"]) - lse_ref))) <= 1e-2


def test_layout_is_validated():
    import ctypes
    import torch
    lib = binding.load()
    shp = binding.FlareShape(1, 1, 8, 32, 16, binding.FLARE_F32, 7)
    f = ctypes.c_size_t(0)
    assert lib.flare_workspace_bytes(ctypes.byref(shp), ctypes.byref(f), None) == -2
    q = torch.zeros((2, 32, 16), device="cuda")
    k = torch.zeros((1, 8, 2, 16), device="cuda")
    with pytest.raises(binding.FlareError):
        binding.forward(q, k, k, 1.0, layout="nhbd")
