"""GPU parity where the geometry of a launch changes: every number of 32-latent tiles with its remainders, chunks of
more than 256 latents that are not whole multiples of anything, and the numbers of token chunks on either side of
where the consumers stop merging the partial slots themselves.

Bars: those of the other parity tests (tests/_util.py): 1e-5 for fp32, 2e-2 with 16-bit storage.
"""
import pytest
import torch

from paper_2508_12594_amd import binding, synth
from tests._util import slice_relerr, to_device, to_host, tol_for

pytestmark = pytest.mark.gpu

# 3, 4 (ragged), 5, 6, 7, 8 tiles; two chunks of 5 and 7; three of 6; d = 16 with fewer tokens than latents
TILES = [(M, d, 700) for M in (65, 96, 97, 130, 161, 192, 200, 225) for d in (8, 16, 32)]
TILES += [(M, d, 1100) for M in (257, 300, 420, 545) for d in (4, 8, 16, 32)] + [(300, 16, 90), (161, 16, 100)]
# H = 1: 1024 tokens per chunk at d = 16, so 16 and 17 slots; short ones with the slots made up to four and eight; fp32: a chunk per 128 tokens
SLOTS = [("bf16", 16 * 1024, 64, 16), ("f16", 16 * 1024 + 1, 64, 16), ("bf16", 16 * 1024 + 1, 64, 8),
         ("bf16", 511, 64, 16), ("bf16", 512, 64, 16), ("f16", 1025, 60, 16), ("bf16", 5000, 33, 8), ("bf16", 140, 256, 32),
         ("bf16", 8 * 1024 + 1, 96, 32), ("f32", 2048, 48, 16), ("f32", 2049, 48, 16), ("f32", 1900, 40, 32)]
# many slots, merged by workgroups of 64 / d latents: one, 3, 8, 9, 17 and 33 of them (neighbours go to one XCD)
SLOTS += [("bf16", 20000, 2, 16), ("f16", 20000, 33, 4), ("bf16", 20000, 16, 32), ("f32", 20000, 65, 8), ("bf16", 40000, 65, 16), ("f32", 5000, 65, 32)]

# fp32: remainders of a tile, the last number of latents whose planes fit in LDS together and the first that runs in
# chunks (d = 8, 16, 32: 256; a token batch is then 1024 tokens in the decode, 512 in dK/dV), more than 2048 latents
F32 = [(33, 4, 129), (31, 8, 33), (97, 16, 260), (160, 32, 257), (256, 16, 1000), (257, 16, 1025), (289, 32, 2049),
       (600, 8, 1100), (2049, 16, 90)]


# numbers of (b,h) that do not divide the chip's workgroups: 3 x 8, 7 x 4, 5 x 4; and more than one per CU
HEADS = [("bf16", 3, 8, 5100, 72, 8), ("f16", 7, 4, 5300, 64, 16), ("bf16", 5, 4, 2700, 130, 32), ("f32", 12, 4, 900, 70, 8),
         ("bf16", 17, 16, 1111, 33, 16), ("f32", 20, 16, 390, 40, 16)]
# more than one round of workgroups: 9 x 16 in every kernel; fp32 chunks of at most 8192 tokens, more than fill the chip
HEADS += [("bf16", 9, 16, 2600, 40, 16), ("f16", 9, 16, 1900, 130, 32), ("f32", 9, 16, 2100, 33, 16), ("f32", 2, 16, 132000, 33, 8)]
# dZ merged by workgroups of two row blocks (2048 of one or more), the last with one
HEADS += [("bf16", 1, 8, 9000, 1025, 16), ("f32", 1, 8, 5000, 513, 32)]


def _check(oracle, dtype, H, N, M, d, layout, saved, B=1):
    print("[case] %s B=%d H=%d N=%d M=%d d=%d %s saved=%s" % (dtype, B, H, N, M, d, layout, saved), flush=True)
    inp = synth.make_inputs(1, B=B, H=H, N=N, M=M, d=d, dtype=dtype, with_dy=True, seed=31 + N + M + d)
    scale, tol, dev = inp["scale"], tol_for(inp), to_device(inp)
    order = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
    k, v, dy = (order(dev[n]) for n in ("k", "v", "dy"))
    ld = torch.empty((B, H, N), dtype=torch.float32, device="cuda") if saved else None
    y, z, lse = binding.forward(dev["q"], k, v, scale, lse_dec=ld, layout=layout)
    dq, dk, dv = binding.backward(dev["q"], k, v, dy, z, lse, scale, y=y if saved else None, lse_dec=ld, layout=layout)
    y_ref, z_ref, _ = oracle.forward(inp["q"], inp["k"], inp["v"], scale)
    dq_ref, dk_ref, dv_ref = oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)
    errs = dict(y=slice_relerr(to_host(order(y)), y_ref), z=slice_relerr(to_host(z), z_ref),
                dq=slice_relerr(to_host(dq), dq_ref), dk=slice_relerr(to_host(order(dk)), dk_ref),
                dv=slice_relerr(to_host(order(dv)), dv_ref))
    print("[case]    " + "  ".join("%s %.2e" % kv for kv in errs.items()), flush=True)
    assert max(errs.values()) <= tol


@pytest.mark.parametrize("M,d,N", TILES)
def test_latent_tiles(oracle, M, d, N):
    _check(oracle, "f16" if M % 3 == 0 else "bf16", 2, N, M, d, "bnhd" if M % 2 else "bhnd", saved=M % 5 != 0)


# fp32 storage, dQ out of the dK/dV kernel (d <= 16, at most 256 latents): one wave to a token tile up to 128 latents, two from
# 129 on (an odd number of tiles between them too), fewer tiles of tokens than waves, one round of them and eight
FUSED_F32 = [(1, 4, 40), (32, 16, 31), (33, 8, 65), (128, 16, 700), (129, 16, 700), (161, 8, 300), (255, 4, 257), (256, 8, 64),
             (160, 16, 9000), (256, 16, 2049), (200, 8, 60000)]


@pytest.mark.parametrize("M,d,N", FUSED_F32)
def test_fused_dq_of_fp32_storage(oracle, M, d, N):
    """Every way to the gradients meets the bar: dQ from the dK/dV kernel (one and two exponentials) and from its own."""
    layout = "bnhd" if N % 2 else "bhnd"
    print("[case] f32 fused dQ N=%d M=%d d=%d %s" % (N, M, d, layout), flush=True)
    inp = synth.make_inputs(1, B=2, H=2, N=N, M=M, d=d, dtype="f32", with_dy=True, seed=5 + N + M + d)
    scale, dev = inp["scale"], to_device(inp)
    order = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
    k, v, dy = (order(dev[n]) for n in ("k", "v", "dy"))
    ld = torch.empty((2, 2, N), dtype=torch.float32, device="cuda")
    y, z, lse = binding.forward(dev["q"], k, v, scale, lse_dec=ld, layout=layout)
    refs = oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)
    for variant in (0, binding.VARIANT_TWO_EXP, binding.VARIANT_SEPARATE_DQ):
        dq, dk, dv = binding.backward(dev["q"], k, v, dy, z, lse, scale, y=y, lse_dec=ld, layout=layout, variant=variant)
        again = binding.backward(dev["q"], k, v, dy, z, lse, scale, y=y, lse_dec=ld, layout=layout, variant=variant)
        errs = [slice_relerr(to_host(g), r) for g, r in zip((dq, order(dk), order(dv)), refs)]
        print("[case]    variant %d: dq %.2e dk %.2e dv %.2e" % ((variant,) + tuple(errs)), flush=True)
        assert max(errs) <= tol_for(inp)
        assert all(torch.equal(a, b) for a, b in zip((dq, dk, dv), again))


@pytest.mark.parametrize("M,d,N", F32)
def test_latent_tiles_of_fp32_storage(oracle, M, d, N):
    _check(oracle, "f32", 2, N, M, d, "bnhd" if M % 2 else "bhnd", saved=M % 3 != 0)


@pytest.mark.parametrize("dtype,N,M,d", SLOTS)
def test_slots_merged_by_consumer_or_kernel(oracle, dtype, N, M, d):
    _check(oracle, dtype, 1, N, M, d, "bhnd", saved=True)


@pytest.mark.parametrize("dtype,B,H,N,M,d", HEADS)
def test_heads_that_do_not_divide_the_chip(oracle, dtype, B, H, N, M, d):
    _check(oracle, dtype, H, N, M, d, "bnhd" if M % 2 else "bhnd", saved=True, B=B)


# d = 32: dQ out of the dK/dV kernel, with all latents in a wave (up to four tiles) or halved between two (three and four
# tiles each, the last ones padding), in chunks of latents; token tiles that leave the last pairs of waves idle or ragged
@pytest.mark.parametrize("M,N,B,layout", [(32, 700, 1, "bhnd"), (128, 1000, 2, "bnhd"), (129, 40, 1, "bhnd"),
                                          (190, 33, 3, "bnhd"), (224, 2049, 1, "bnhd"), (256, 130, 2, "bhnd"),
                                          (256, 4100, 1, "bhnd"), (330, 1000, 1, "bnhd")])
def test_fused_dq_of_wide_heads(oracle, M, N, B, layout):
    """Against the oracle and against the dQ kernel of its own."""
    _check(oracle, "f16" if M == 190 else "bf16", 2, N, M, 32, layout, saved=M != 128, B=B)
    inp = synth.make_inputs(1, B=B, H=2, N=N, M=M, d=32, dtype="bf16", with_dy=True, seed=3 + N + M)
    dev = to_device(inp)
    y, z, lse = binding.forward(dev["q"], dev["k"], dev["v"], inp["scale"])
    one, two = (binding.backward(dev["q"], dev["k"], dev["v"], dev["dy"], z, lse, inp["scale"], variant=x)
                for x in (0, binding.VARIANT_SEPARATE_DQ))
    for a, b in zip(one, two):
        assert slice_relerr(to_host(a), to_host(b)) <= tol_for(inp)


@pytest.mark.parametrize("dtype,M,N,d", [("bf16", 32, 300, 32), ("f16", 90, 515, 32), ("bf16", 128, 1000, 32), ("bf16", 190, 333, 32),
                                         ("bf16", 256, 1100, 32), ("f16", 330, 700, 32), ("bf16", 336, 1000, 16)])
def test_two_exponentials_in_the_fused_kernel(oracle, dtype, M, N, d):
    """The form that inputs with far log-sum-exps take, at every way to hold the latents."""
    inp = synth.make_inputs(1, B=2, H=2, N=N, M=M, d=d, dtype=dtype, with_dy=True, seed=5 + N + M)
    dev, scale, tol = to_device(inp), inp["scale"], tol_for(inp)
    ld = torch.empty((2, 2, N), dtype=torch.float32, device="cuda")
    y, z, lse = binding.forward(dev["q"], dev["k"], dev["v"], scale, lse_dec=ld)
    got = binding.backward(dev["q"], dev["k"], dev["v"], dev["dy"], z, lse, scale, y=y, lse_dec=ld,
                           variant=binding.VARIANT_TWO_EXP)
    for a, ref in zip(got, oracle.backward(inp["q"], inp["k"], inp["v"], inp["dy"], scale)):
        assert slice_relerr(to_host(a), ref) <= tol


# d = 32, chunks of seven and eight latent tiles: the last number of tokens with a dQ kernel of its own, the first without
@pytest.mark.parametrize("dtype,M,N,layout", [("bf16", 450, 8192, "bhnd"), ("f16", 450, 8193, "bnhd"), ("f16", 385, 65, "bnhd"),
                                              ("bf16", 640, 300, "bhnd")])
def test_few_tokens_beside_chunks_of_wide_latents(oracle, dtype, M, N, layout):
    _check(oracle, dtype, 2, N, M, 32, layout, saved=True)


# the decode of more than 256 latents, chunk after chunk: chunks whose scores lie far above or below those so far, the last
# one all but empty, tokens behind the last whole tile, both types of y
@pytest.mark.parametrize("M,d,N,layout,y_f32,gains", [
    (257, 8, 95, "bhnd", True, (1, 60)), (300, 16, 333, "bnhd", False, (60, 1)), (545, 4, 1000, "bhnd", False, (1, 60, 1)),
    (768, 16, 64, "bhnd", True, (60, 1, 20)), (1030, 8, 700, "bnhd", False, (1, 5, 40, 1, 80)), (300, 32, 333, "bhnd", True, (60, 1))])
def test_decode_of_chunks_far_apart(M, d, N, layout, y_f32, gains):
    """Against the softmax in 64 bits."""
    print("[case] decode M=%d d=%d N=%d" % (M, d, N), flush=True)
    inp = synth.make_inputs(1, B=2, H=2, N=N, M=M, d=d, dtype="bf16", seed=M + N)
    dev = to_device(inp, ("q", "k", "v"))
    step = 32 * -(-(-(-M // 32)) // len(gains))
    gain = torch.cat([torch.full((step,), float(g)) for g in gains])[:M].to("cuda")
    q = (dev["q"] * gain[:, None]).to(dev["q"].dtype)
    k, v = (t.permute(0, 2, 1, 3).contiguous() if layout == "bnhd" else t for t in (dev["k"], dev["v"]))
    ld = torch.empty((2, 2, N), dtype=torch.float32, device="cuda")
    y, z, _ = binding.forward(q, k, v, inp["scale"], lse_dec=ld, layout=layout, y_f32=y_f32)
    y = y.permute(0, 2, 1, 3) if layout == "bnhd" else y
    s = torch.matmul(dev["k"].double().cpu(), q.double().cpu().transpose(1, 2)) * inp["scale"]
    y_ref = torch.matmul(s.softmax(-1), z.double().cpu())
    assert slice_relerr(to_host(y), y_ref.numpy()) <= tol_for(inp)
    # log-sums: queries as a pair of bf16 terms (2^-16 of a score's terms), weights rounded to bf16 (2^-9)
    terms = torch.matmul(dev["k"].double().cpu().abs(), q.double().cpu().abs().transpose(1, 2)).amax(-1) * inp["scale"]
    assert ((ld.double().cpu() - s.logsumexp(-1)).abs() <= 2.0 ** -16 * terms + 2.0 ** -8).all()


@pytest.mark.parametrize("M", [70, 150, 200])
def test_projection_of_ragged_latents(M):
    """The fused projection forms the y that the decode forms, bit for bit, whatever the number of tiles."""
    print("[case] projection M=%d" % M, flush=True)
    inp = synth.make_inputs(1, B=1, H=4, N=777, M=M, d=16, dtype="bf16", seed=5 + M)
    dev = to_device(inp, ("q", "k", "v"))
    k, v = (dev[n].permute(0, 2, 1, 3).contiguous() for n in ("k", "v"))
    y_ref, z_ref, lse_ref = binding.forward(dev["q"], k, v, inp["scale"], layout="bnhd")
    y = torch.empty_like(k)
    w = torch.eye(64, dtype=k.dtype, device="cuda")
    out, z, lse = binding.forward_project(dev["q"], k, v, w, inp["scale"], y=y)
    assert torch.equal(z, z_ref) and torch.equal(lse, lse_ref)
    # (z that the decode merged for itself and z from memory are the same numbers)
    assert torch.equal(y, y_ref) and torch.equal(out.view_as(y), y)


@pytest.mark.parametrize("B,H", [(11, 8), (7, 4), (5, 2)])
def test_projection_of_items_that_do_not_divide_the_chip(B, H):
    print("[case] projection B=%d H=%d" % (B, H), flush=True)
    inp = synth.make_inputs(1, B=B, H=H, N=1111, M=50, d=16, dtype="bf16", seed=5 + B)
    dev = to_device(inp, ("q", "k", "v"))
    k, v = (dev[n].permute(0, 2, 1, 3).contiguous() for n in ("k", "v"))
    y_ref = binding.forward(dev["q"], k, v, inp["scale"], layout="bnhd")[0]
    w = torch.eye(16 * H, dtype=k.dtype, device="cuda")
    out = binding.forward_project(dev["q"], k, v, w, inp["scale"])[0]
    assert torch.equal(out.view_as(y_ref), y_ref)
