"""Timed cases of the FLARE token mixer: what a program that uses this package has it do, from the smallest calls
to the largest, through the public entry points.

A case is a dict of plain values:
  op      "train":   flare_mixer(...) and the gradients of q_lat, k and v (a layer inside a model, torch.autograd)
          "step":    binding.forward and binding.backward with buffers the program keeps (a hand-written training loop)
          "forward": binding.forward with nothing kept (inference)
          "project": binding.forward_project, the forward with the block's output projection (inference)
          "static":  binding.forward_static into buffers the program keeps (a serving loop)
  B, H, N, M, d    batch items, heads, tokens per item, latent queries per head, head dimension
  dtype   "bf16", "f16" (the autocast type) or "f32"
  layout  order of the token tensors: "bhnd" or "bnhd" (what a block's linear layers write)
  inputs  "mesh" (smooth fields on random points, lifted and projected to keys and values: a PDE surrogate) or
          "normal" (sequence features behind a normalisation)
  y_f32   whether the mixer hands y over in fp32 (a training option for small head dimensions)
"""
import math

import torch

from paper_2508_12594_amd import binding
from paper_2508_12594_amd.autograd import flare_mixer

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _case(name, op, B, H, N, M, d, dtype, layout="bhnd", inputs="mesh", y_f32=False):
    c = dict(op=op, B=B, H=H, N=N, M=M, d=d, dtype=dtype, layout=layout, inputs=inputs, y_f32=y_f32)
    return dict(c, name=name) if name else c


def listed():
    return [
        # One small mesh at a time in a serving loop: the smallest call, nothing but latency.
        _case("serve-small-mesh", "static", 1, 8, 1024, 64, 16, "bf16"),
        # Single-precision training on one short sequence (the first reference workload).
        _case("train-f32-short", "train", 1, 4, 1024, 64, 32, "f32", inputs="normal"),
        # Two 85 x 85 grids per step under fp16 autocast, in the order the K/V projections write; ragged N and M.
        _case("train-f16-grid", "train", 2, 8, 7225, 100, 16, "f16", layout="bnhd"),
        # A batch of 2-D meshes (the second reference workload).
        _case("train-bf16-meshes", "train", 4, 8, 16384, 64, 16, "bf16"),
        # A batch of 4k-token sequences for classification (the third reference workload).
        _case("train-bf16-sequences", "train", 32, 8, 4096, 128, 32, "bf16", inputs="normal"),
        # Single-precision inference on a mesh of an odd number of points.
        _case("infer-f32-mesh", "forward", 1, 8, 30011, 128, 16, "f32"),
        # Single-precision training on a large mesh.
        _case("train-f32-mesh", "train", 1, 8, 100000, 256, 16, "f32"),
        # Inference on a small batch of large meshes with the narrow heads of a C = 64 model; ragged N and M.
        _case("infer-bf16-narrow", "forward", 3, 8, 50021, 200, 8, "bf16", layout="bnhd"),
        # Long sequences with wide heads (the fifth reference workload).
        _case("train-bf16-long", "train", 1, 8, 262144, 256, 32, "bf16", inputs="normal"),
        # Inference of a block's mixer with its output projection on a million points.
        _case("project-bf16-million", "project", 1, 8, 1000000, 256, 16, "bf16", layout="bnhd"),
        # One training step on a million points (the fourth reference workload, bench.py's default).
        _case("step-bf16-million", "step", 1, 8, 1000000, 256, 16, "bf16"),
        # The largest model of the million-point study: 2048 latents, C = 64.
        _case("train-bf16-2048-latents", "train", 1, 8, 1000000, 2048, 8, "bf16", y_f32=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over their whole range (logarithmically), mostly not multiples of anything."""
    op = rng.choice(["train", "train", "train", "step", "forward", "forward", "project", "static"])
    dtype = rng.choice(["bf16", "bf16", "f16"] if op == "project" else ["bf16", "bf16", "bf16", "f16", "f32", "f32"])
    H = rng.choice([4, 8]) if op == "project" else rng.choice([4, 8, 8, 16])
    d = 16 if op == "project" else rng.choice([8, 16, 16, 32])
    layout = "bnhd" if op == "project" else rng.choice(["bhnd", "bhnd", "bnhd"])
    B = 1 if op == "static" else rng.choice([1, 1, 1, 2, 4, _log_uniform(rng, 1, 32)])
    if op == "static":       # a serving loop's scratch is the library's own 32 MiB
        N, M = _log_uniform(rng, 512, 8192), _log_uniform(rng, 16, 128)
    else:
        N = _log_uniform(rng, 512, 1000000 // B)
        M = _log_uniform(rng, 16, 256 if op == "project" else 512 if dtype == "f32" else 2048)
    if rng.random() < 0.4:   # models use round numbers of latents; ragged ones come from ablations
        M = min(max(16, 1 << round(math.log2(M))), 256 if op == "project" else 2048)
    # no more work than the largest listed case (single precision costs about ten times as much a score)
    most = (8e8 if dtype == "f32" else 1.6e10) * min(1.0, 8 / d if dtype != "f32" else 16 / d)
    N = max(512, min(N, int(most / (B * H * M))))
    y_f32 = op == "train" and dtype != "f32" and d == 8 and rng.random() < 0.5
    return _case(None, op, B, H, N, M, d, dtype, layout, rng.choice(["mesh", "mesh", "normal"]), y_f32)


def _token_inputs(c, gen):
    """Keys and values [B,H,N,d] (fp32) with the statistics of a layer's projections."""
    B, H, N, d = c["B"], c["H"], c["N"], c["d"]
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda")   # noqa: E731
    if c["inputs"] == "normal":
        return randn(B, H, N, d), randn(B, H, N, d)
    C = H * d
    points = torch.rand((B, N, 3), generator=gen, device="cuda")
    waves = torch.randint(1, 4, (B, 3, 3), generator=gen, device="cuda").float()
    phase = torch.rand((B, 1, 3), generator=gen, device="cuda") * (2 * math.pi)
    fields = torch.sin(2 * math.pi * torch.matmul(points, waves) + phase)
    features = torch.matmul(torch.cat([points, fields], 2), randn(B, 6, C))
    features += 0.1 * randn(B, N, C)
    out = []
    for _ in range(2):
        w = randn(C, C) / math.sqrt(C)
        out.append(torch.matmul(features.view(B * N, C), w).view(B, N, H, d).transpose(1, 2).contiguous())
    return out


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, H, N, M, d = (c[x] for x in "BHNMd")
    dt, layout = DTYPES[c["dtype"]], c["layout"]
    order = (lambda t: t) if layout == "bhnd" else (lambda t: t.transpose(1, 2))
    k, v = _token_inputs(c, gen)
    s = dict(c, scale=1.0 / math.sqrt(d))
    s["q"] = torch.randn((H, M, d), generator=gen, device="cuda").to(dt)
    s["k"], s["v"] = (order(t).to(dt).contiguous() for t in (k, v))
    del k, v
    f32 = dict(dtype=torch.float32, device="cuda")
    if c["op"] in ("train", "step"):     # the loss's gradient comes back in the type of y
        dy = torch.randn(s["k"].shape, generator=gen, device="cuda").to(dt)
        s["dy"] = dy.float() if c["y_f32"] else dy
    if c["op"] == "train":
        for n in ("q", "k", "v"):
            s[n].requires_grad_(True)
    if c["op"] in ("step", "static"):    # buffers that the program keeps
        s["y"] = torch.empty_like(s["k"])
        s["z"] = torch.empty((B, H, M, d), **f32)
        s["lse_enc"] = torch.empty((B, H, M), **f32)
    if c["op"] == "step":
        s["lse_dec"] = torch.empty((B, H, N), **f32)
        s["dq"] = torch.empty((H, M, d), **f32)
        s["dk"], s["dv"] = torch.empty_like(s["k"]), torch.empty_like(s["k"])
        code = {"bf16": binding.FLARE_BF16, "f16": binding.FLARE_F16, "f32": binding.FLARE_F32}[c["dtype"]]
        s["workspace"] = torch.empty(max(256, *binding.workspace_bytes(B, H, N, M, d, code)), dtype=torch.uint8,
                                     device="cuda")
    if c["op"] == "project":
        C = H * d
        s["w_out"] = (torch.randn((C, C), generator=gen, device="cuda") / math.sqrt(C)).to(dt)
        s["bias"] = 0.1 * torch.randn((C,), generator=gen, device="cuda")
    return s


def run(s):
    op, q, k, v, scale, layout = s["op"], s["q"], s["k"], s["v"], s["scale"], s["layout"]
    if op == "train":
        y = flare_mixer(q, k, v, scale, layout=layout, y_f32=s["y_f32"])
        dq, dk, dv = torch.autograd.grad(y, (q, k, v), s["dy"])
        return {"y": y, "dq": dq, "dk": dk, "dv": dv}
    if op == "forward":
        y, z, lse_enc = binding.forward(q, k, v, scale, layout=layout)
        return {"y": y, "z": z, "lse_enc": lse_enc}
    if op == "project":
        out, z, lse_enc = binding.forward_project(q, k, v, s["w_out"], scale, bias=s["bias"])
        return {"out": out, "z": z, "lse_enc": lse_enc}
    if op == "static":
        y, z, lse_enc = binding.forward_static(q, k, v, scale, s["y"], s["z"], s["lse_enc"], layout=layout)
        return {"y": y, "z": z, "lse_enc": lse_enc}
    y, z, lse_enc = binding.forward(q, k, v, scale, y=s["y"], z=s["z"], lse_enc=s["lse_enc"], lse_dec=s["lse_dec"],
                                    workspace=s["workspace"], layout=layout)
    dq, dk, dv = binding.backward(q, k, v, s["dy"], z, lse_enc, scale, y=y, lse_dec=s["lse_dec"], dq_lat=s["dq"],
                                  dk=s["dk"], dv=s["dv"], workspace=s["workspace"], layout=layout)
    return {"y": y, "z": z, "lse_enc": lse_enc, "dq": dq, "dk": dk, "dv": dv}


def work(case):
    B, H, N, M, d = (case[x] for x in "BHNMd")
    elem = 4 if case["dtype"] == "f32" else 2
    y_elem = 4 if case["y_f32"] else elem
    tok, lat = B * H * N * d, B * H * M * d
    product = 2.0 * B * H * N * M * d           # one contraction over the scores of every head
    bytes_ = tok * (2 * elem + y_elem) + H * M * d * elem      # k, v; y; q_lat
    flops = 3 * product                         # the scores, encode, decode
    if case["op"] != "train":
        bytes_ += 4 * (lat + B * H * M)         # z, lse_enc
    if case["op"] in ("train", "step"):         # dy; dk, dv; dq_lat
        bytes_ += tok * (y_elem + 2 * elem) + H * M * d * (elem if case["op"] == "train" else 4)
        flops += 6 * product                    # dZ, <dZ, V>, <Z, dY>, dV, dK, dQ
    if case["op"] == "project":
        C = H * d
        bytes_ += C * C * elem + 4 * C
        flops += 2.0 * B * N * C * C
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """Sums of up to a million 32-bit terms agree to 1e-5, gradients (differences of such sums) to twice that.  With
    16-bit storage the softmax weights are rounded to bf16 (2^-9, independent), and gradients, again differences of
    sums of such terms, show several times that."""
    backward = case["op"] in ("train", "step")
    if case["dtype"] == "f32":
        return {"rel": 2e-5 if backward else 1e-5}
    return {"rel": 2e-2 if backward else 1e-2}
