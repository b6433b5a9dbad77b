"""fp32 storage where the scores, the values or the gradients lie far from one: the forms of the matrix-core kernels that
ordinary inputs do not reach (a running maximum, exact maxima per token, both exponentials of the backward), at ragged
sizes.  Reference: the fp64 oracle.

Bounds.  A score of S2 log2 units is rounded by |S2| 2^-24, which multiplies its weight, beside the 1e-5 of the fp32 path:
y, z and dV are held to 1e-5 + |S2| 2^-23 (a score is a sum of six plane products, so it is rounded more than once).  dQ and
dK are differences of terms K times as large (see test_gpu_fp32_conditioning.py): 1e-5 + (8 + |S2|) 2^-24 K.
"""
import numpy as np
import pytest
import torch

from paper_2508_12594_amd import binding, synth
from tests._util import slice_relerr, to_device, to_host
from tests.test_gpu_fp32_conditioning import LOG2E, _cancellation_factor

pytestmark = pytest.mark.gpu


def _inputs(N, M, d, seed=0):
    return synth.make_inputs(1, B=1, H=2, N=N, M=M, d=d, dtype="f32", with_dy=True, seed=41 + seed + N + M + d)


def _shift_scores(inp, nats):
    """All scores of head 1 move by the same amount: a first query coordinate of 8 (exact products, and at the magnitude
    of the other queries' sum), and the first key coordinate that gives it."""
    q, k = inp["q"].copy(), inp["k"].copy()
    q[1, :, 0] = 8.0
    k[:, 1, :, 0] = np.float32(nats / (8.0 * inp["scale"]))
    return dict(inp, q=q, k=k)


def _check(oracle, inp, saved, layout="bhnd", variant=0):
    scale, dev = inp["scale"], to_device(inp)
    order = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
    k, v, dy = (order(dev[n]) for n in ("k", "v", "dy"))
    ld = torch.empty(dev["k"].shape[:3], dtype=torch.float32, device="cuda") if saved else None
    y, z, lse = binding.forward(dev["q"], k, v, scale, lse_dec=ld, layout=layout)
    dq, dk, dv = binding.backward(dev["q"], k, v, dy, z, lse, scale, y=y if saved else None, lse_dec=ld, layout=layout,
                                  variant=variant)
    y_ref, z_ref, _ = oracle.forward(inp["q"], inp["k"], inp["v"], scale)
    refs = oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)
    got = dict(y=order(y), z=z, dq=dq, dk=order(dk), dv=order(dv))
    for h in range(inp["q"].shape[0]):
        one = lambda t: t[h:h + 1] if t.ndim == 3 else t[:, h:h + 1]   # noqa: E731
        part = {n: one(inp[n]) for n in ("q", "k", "v", "dy")}
        s2 = float(np.max(np.abs(np.einsum("hmj,bhnj->bhmn", part["q"], part["k"])))) * scale * LOG2E
        ref = dict(zip(("y", "z", "dq", "dk", "dv"), map(one, (y_ref, z_ref) + tuple(refs))))
        K, K_dk = _cancellation_factor(part["q"], part["k"], part["v"], part["dy"], scale, ref["dq"], ref["dk"])
        bound = dict.fromkeys(("y", "z", "dv"), 1e-5 + s2 * 2.0 ** -23)
        bound.update(dq=1e-5 + (8 + s2) * 2.0 ** -24 * K, dk=1e-5 + (8 + s2) * 2.0 ** -24 * K_dk)
        host = {n: one(to_host(t)) for n, t in got.items()}
        errs = {n: slice_relerr(host[n], ref[n]) for n in host}
        print("[case]    head %d, |S2| to %.0f, K %.0f %.0f: " % (h, s2, K, K_dk) +
              "  ".join("%s %.2e (%.1e)" % (n, errs[n], bound[n]) for n in errs), flush=True)
        for n in errs:
            assert np.isfinite(host[n]).all(), n
            assert errs[n] <= bound[n], n


# one chunk of latents whose slots the consumers merge, the same merged by kernels of their own (N = 3001: more slots than
# that), and latents in chunks; every head dimension's staging
SHAPES = [(1001, 64, 16), (3001, 96, 8), (1001, 300, 16), (700, 300, 8), (515, 40, 32), (1030, 320, 32), (333, 33, 4)]


@pytest.mark.parametrize("saved", [True, False])
@pytest.mark.parametrize("N,M,d", SHAPES)
@pytest.mark.parametrize("nats", [-150.0, -45.0, 45.0, 150.0])
def test_every_score_shifted(oracle, nats, N, M, d, saved):
    """log-sum-exps far below and far above zero, where 2^-lse or 2^S alone is no fp32 number, and just beyond the span in
    which the kernels work without a normaliser; head 0 stays ordinary."""
    print("[case] fp32, scores of one head shifted by %g: N=%d M=%d d=%d saved=%s" % (nats, N, M, d, saved), flush=True)
    _check(oracle, _shift_scores(_inputs(N, M, d), nats), saved, layout="bnhd" if M == 96 else "bhnd")


@pytest.mark.parametrize("saved", [True, False])
@pytest.mark.parametrize("M,d", [(64, 16), (300, 8), (128, 32)])
def test_wide_score_range(oracle, M, d, saved):
    """Head 1 has latents whose score offsets are hundreds of log2 units apart, so that no one stabiliser fits them all."""
    print("[case] fp32, wide score range: M=%d d=%d saved=%s" % (M, d, saved), flush=True)
    inp = _inputs(1500, M, d)
    q, k = inp["q"].copy(), inp["k"].copy()
    k[:, 1, :, 0] = 4.0
    q[1, :, 0] = np.linspace(-120.0, 120.0, M, dtype=np.float32) * np.float32(0.25 / inp["scale"])
    _check(oracle, dict(inp, q=q, k=k), saved)


# Weights are summed as 2^S while nothing leaves the range of fp32 that way: scores within that range, and values or
# gradients large or small enough that 2^S times them is not.
@pytest.mark.parametrize("N,M,d", SHAPES)
@pytest.mark.parametrize("nats,v_size,dy_size", [(61.0, 1e12, 1.0), (25.0, 1e25, 1e-18), (-55.0, 1e-21, 1.0),
                                                 (-40.0, 1.0, 1e-20), (38.0, 1.0, 1e-20), (18.0, 1.0, 1e-20)])
def test_size_of_values_and_gradients(oracle, nats, v_size, dy_size, N, M, d):
    print("[case] fp32, scores shifted by %g, v of %g, dY of %g: N=%d M=%d d=%d" % (nats, v_size, dy_size, N, M, d), flush=True)
    inp = _shift_scores(_inputs(N, M, d), nats)
    inp = dict(inp, v=inp["v"] * np.float32(v_size), dy=inp["dy"] * np.float32(dy_size))
    _check(oracle, inp, saved=N > 600)


@pytest.mark.parametrize("N,M,d", SHAPES)
def test_two_exponential_kernels(oracle, N, M, d):
    """The two-exponential form of the backward, forced on ordinary inputs."""
    print("[case] fp32, two exponentials forced: N=%d M=%d d=%d" % (N, M, d), flush=True)
    _check(oracle, _inputs(N, M, d), saved=N != 515, variant=binding.VARIANT_TWO_EXP)


# Rounding to nearest averages out over the terms of a sum; an error of one sign does not.  With independent roundings the
# weights are good to a few 2^-24 (|S2| below 10 here), and means of values and gradients under them no worse: 8 * 2^-24.
# (The logarithm's one-sided cut and a rounded lse log2 e gave dV 8e-7 ... 1.2e-6 on these inputs, small accumulators that the
# matrix cores cut downwards y 4.7e-7 and dV another 3e-7 on the first.)
UNBIASED = 8 * 2.0 ** -24


@pytest.mark.parametrize("kind,N,M,d", [(1, 100000, 64, 32), (1, 60000, 256, 16), (4, 2485, 128, 16), (2, 20000, 32, 8)])
def test_roundings_average_out(oracle, kind, N, M, d):
    """Sums over many tokens: mean-zero values (kind 1), whose mean is small, and mesh-like ones."""
    print("[case] fp32, unbiased sums: kind %d N=%d M=%d d=%d" % (kind, N, M, d), flush=True)
    inp = synth.make_inputs(kind, B=1, H=2, N=N, M=M, d=d, dtype="f32", with_dy=True, seed=71 + N)
    dev, scale = to_device(inp), inp["scale"]
    ld = torch.empty((1, 2, N), dtype=torch.float32, device="cuda")
    y, z, lse = binding.forward(dev["q"], dev["k"], dev["v"], scale, lse_dec=ld)
    dq, dk, dv = binding.backward(dev["q"], dev["k"], dev["v"], dev["dy"], z, lse, scale, y=y, lse_dec=ld)
    y_ref, _, lse_ref = oracle.forward(inp["q"], inp["k"], inp["v"], scale)
    dv_ref = oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)[2]
    err = lse.double().cpu().numpy() - lse_ref
    print("[case]    y %.2e dv %.2e; lse_enc mean error %.1e" % (slice_relerr(to_host(y), y_ref),
                                                                slice_relerr(to_host(dv), dv_ref), err.mean()), flush=True)
    assert slice_relerr(to_host(y), y_ref) <= UNBIASED and slice_relerr(to_host(dv), dv_ref) <= UNBIASED
    assert abs(err.mean()) <= 2.0 ** -22     # rounded to nearest its mean vanishes; half an ulp of 8 ... 16 is 2^-21


@pytest.mark.parametrize("B,N,M,d", [(60, 4930, 4, 16), (12, 3410, 2, 16), (4, 6019, 14, 32), (8, 1500, 300, 8)])
def test_keys_far_from_their_spread(oracle, B, N, M, d):
    """Keys whose common part is many times what tells them apart: the terms of dQ are K times as large as their sum, and eps
    and the normalisers, rounded to 2^-24, enter them: 8 * 2^-24 K as in test_gpu_fp32_conditioning.py, with nothing for an
    error that all tokens share."""
    print("[case] fp32, long common key: B=%d N=%d M=%d d=%d" % (B, N, M, d), flush=True)
    inp = synth.make_inputs(1, B=B, H=1, N=N, M=M, d=d, dtype="f32", with_dy=True, seed=5 + N)
    common = np.random.Generator(np.random.PCG64(N)).standard_normal(d).astype(np.float32)
    inp["k"] = np.float32(0.3) * inp["k"] + np.float32(2.0) * common
    dev, scale = to_device(inp), inp["scale"]
    refs = oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)
    K = _cancellation_factor(inp["q"], inp["k"], inp["v"], inp["dy"], scale, refs[0])
    for saved in (True, False):
        ld = torch.empty((B, 1, N), dtype=torch.float32, device="cuda") if saved else None
        y, z, lse = binding.forward(dev["q"], dev["k"], dev["v"], scale, lse_dec=ld)
        dq, _, _ = binding.backward(dev["q"], dev["k"], dev["v"], dev["dy"], z, lse, scale, y=y if saved else None, lse_dec=ld)
        e = slice_relerr(to_host(dq), refs[0])
        print("[case]    saved=%s dq %.2e, K %.0f: bound %.2e" % (saved, e, K, UNBIASED + 8 * 2.0 ** -24 * K), flush=True)
        assert e <= UNBIASED + 8 * 2.0 ** -24 * K
