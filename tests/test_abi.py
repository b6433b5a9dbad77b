"""The C-ABI library loads, exports every symbol include/flare.h declares, and rejects bad
arguments on the host before anything is launched (no GPU needed, no compute calls)."""
import ctypes
import os
import re

import pytest

from paper_2508_12594_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2508_12594_amd import build
        build.build_library(verbose=False)
    return binding.load()


def _declared(header):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return set(re.findall(r"\b(flare_[a-z_]+)\s*\(", text))


def test_header_symbols_are_exported(lib):
    """Every function an include/*.h declares is exported by the library it belongs to, and the bindings
    list exactly those: flare.h (the operator) and flare_profile.h (timing hooks) -> libflare.so,
    flare_rates.h (machine-rate micro-benchmarks) -> libflare_rates.so."""
    headers = sorted(f for f in os.listdir(os.path.join(ROOT, "include")) if f.endswith(".h"))
    assert headers == ["flare.h", "flare_profile.h", "flare_rates.h"]
    declared = sorted(_declared("flare.h") | _declared("flare_profile.h"))
    assert declared == sorted(binding.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name
    from paper_2508_12594_amd import rates
    rl = rates.load()
    assert sorted(_declared("flare_rates.h")) == sorted(rates.EXPORTS)
    for name in rates.EXPORTS:
        assert hasattr(rl, name), name
    assert rl.flare_rates_count() == len(rates.names()) > 10


def test_version_and_strerror(lib):
    assert binding.version() >= 200
    assert binding.strerror(0) == "success"
    for code in (-1, -2, -3, -4, -5, -6, -99):
        assert len(binding.strerror(code)) > 0


def test_workspace_bytes_of_any_shape(lib):
    """Shapes far beyond any memory are answered like others (a crash here would take the program with it)."""
    for dtype in (binding.FLARE_F32, binding.FLARE_BF16):
        for B, H, N, M, d in ((65535, 1, 100, 1 << 21, 4), (8191, 8, 1000, 1 << 24, 8), (1, 1, 100, (1 << 31) - 1, 4),
                              (60000, 1, 1 << 23, (1 << 22) + 32, 4), (1, 65535, (1 << 24) - 1, 1, 4)):
            f, b = binding.workspace_bytes(B, H, N, M, d, dtype)
            assert f >= B * H * M * (d + 2) * 4 or M == 1
            assert b >= f // 2


@pytest.mark.parametrize("B,H,N,M,d,chunks", [(1, 8, 13407, 44, 32, 105), (1, 16, 12743, 22, 32, 100), (4, 8, 55441, 189, 16, 22),
                                              (1, 4, 119557, 50, 16, 117), (4, 16, 6181, 64, 16, 7), (1, 8, 41742, 40, 16, 55),
                                              (2, 16, 292664, 25, 16, 36)])
def test_fp32_chunks_are_short_enough(lib, B, H, N, M, d, chunks):
    """fp32 sums are taken one after the other over a chunk of tokens (a partial slot each, so the forward's workspace counts
    them): 16 waves on each of the 256 compute units, and no chunk above 8192 tokens, set how long it may be."""
    f, _ = binding.workspace_bytes(B, H, N, M, d, binding.FLARE_F32)
    assert f // (4 * B * H * M * (d + 2)) >= chunks


@pytest.mark.parametrize("B,H,N,M,d", [(2, 8, 6397, 357, 32), (1, 8, 8472, 543, 32), (4, 16, 8983, 1766, 16), (3, 8, 117199, 256, 16),
                                       (1, 16, 12731, 176, 32)])
def test_more_fp32_chunks_still_fit_the_static_scratch(lib, B, H, N, M, d):
    """Taking more chunks than the chip calls for must not make flare_forward_static refuse a shape (32 MiB)."""
    f, _ = binding.workspace_bytes(B, H, N, M, d, binding.FLARE_F32)
    assert f <= 32 << 20


@pytest.mark.parametrize("B,H,N,M,d,slots", [(56, 1, 2285, 136, 32, 24), (5, 8, 3695, 89, 32, 24), (50, 1, 3206, 224, 16, 24),
                                             (14, 4, 2509, 149, 32, 24), (3, 16, 2573, 104, 32, 24)])
def test_backward_workspace_holds_the_slots_that_are_written(lib, B, H, N, M, d, slots):
    """16-bit storage, dZ merged by its consumer (at most 16 slots): beside the per-token statistics and one row per latent the
    workspace holds a few slots of dZ and of dQ, not the vector kernels' 2048 / (B H) of each."""
    _, b = binding.workspace_bytes(B, H, N, M, d, binding.FLARE_BF16)
    assert b - 8 * B * H * N <= (slots + 2) * 4 * B * H * M * d


def test_backward_workspace_serves_the_variants(lib):
    """The size for a shape as it comes is enough for the same shape with a dQ kernel of its own."""
    for dtype in (binding.FLARE_BF16, binding.FLARE_F32):
        for d in (4, 8, 16, 32):
            for M in (33, 128, 129, 200, 256, 257, 300, 450, 2048):
                for N in (16, 300, 5000, 100000):
                    for B, H in ((1, 1), (1, 8), (3, 8), (14, 4), (64, 32)):
                        size = []
                        for variant in (0, binding.VARIANT_SEPARATE_DQ, binding.VARIANT_TWO_EXP):
                            b = ctypes.c_size_t(0)
                            shp = binding.FlareShape(B, H, N, M, d, dtype, 0, 0, 0, variant)
                            assert lib.flare_workspace_bytes(ctypes.byref(shp), None, ctypes.byref(b)) == 0
                            size.append(b.value)
                        assert max(size) == size[0]


@pytest.mark.parametrize("B,H,N", [(64, 32, 1000000), (300, 100, 200000), (16, 16, 3000000), (1, 8, 100000), (1, 1, 16)])
def test_fused_fp32_dq_is_summed_over_few_enough_tokens(lib, B, H, N):
    """Where dQ comes out of the fp32 dK/dV kernel a wave adds up its token tiles one after the other: at most 8192 tokens, however many
    (b,h) fill the chip with few workgroups each; and the workspace holds a slot for each of those workgroups."""
    blocks_of = lib["_ZN5flare16mfma32_dq_blocksERK11flare_shape"]
    tiles = -(-N // 32)
    for d in (4, 8, 16):
        for M in (33, 128, 129, 256):
            shp, b = binding.FlareShape(B, H, N, M, d, binding.FLARE_F32), ctypes.c_size_t(0)
            blocks = blocks_of(ctypes.byref(shp))
            waves = 8 if M <= 128 else 4                    # token tiles a workgroup of eight waves works on at a time
            assert blocks >= 1 and -(-tiles // (blocks * waves)) * 32 <= 8192, (M, d)
            assert lib.flare_workspace_bytes(ctypes.byref(shp), None, ctypes.byref(b)) == 0
            assert b.value >= 4 * B * H * (2 * N + (blocks + 1) * M * d), (M, d)
    shp = binding.FlareShape(B, H, N, 200, 16, binding.FLARE_F32, 0, 0, 0, binding.VARIANT_SEPARATE_DQ)
    assert blocks_of(ctypes.byref(shp)) == 0                # (a dQ kernel of its own)


def test_workspace_bytes_do_not_depend_on_the_layout(lib):
    """binding.workspace_bytes has no layout argument: what it reports has to serve both.  Few tokens, where one slot more
    per chunk is the largest count there is, every tile count and head dimension."""
    def both(*dims):
        out = []
        for layout in (binding.FLARE_BHND, binding.FLARE_BNHD):
            f, b = ctypes.c_size_t(0), ctypes.c_size_t(0)
            shp = binding.FlareShape(*dims, layout)
            assert lib.flare_workspace_bytes(ctypes.byref(shp), ctypes.byref(f), ctypes.byref(b)) == 0
            out.append((f.value, b.value))
        return out

    for dtype in (binding.FLARE_F32, binding.FLARE_BF16, binding.FLARE_F16):
        for d in (4, 8, 16, 32):
            for M in (1, 33, 65, 96, 100, 128, 129, 200, 256, 300, 2048):
                for N in (1, 16, 31, 57, 300, 5000, 100000):
                    for B, H in ((1, 1), (1, 8), (3, 8), (25, 2), (64, 32), (300, 100)):
                        bhnd, bnhd = both(B, H, N, M, d, dtype)
                        assert bhnd == bnhd, (B, H, N, M, d, dtype)
                        assert binding.workspace_bytes(B, H, N, M, d, dtype) == bnhd


def test_workspace_bytes_and_shape_checks(lib):
    f, b = binding.workspace_bytes(1, 8, 1000000, 256, 16, binding.FLARE_BF16)
    assert 0 < f < 64 << 20 and b > 0
    f1, _ = binding.workspace_bytes(1, 4, 1024, 64, 32, binding.FLARE_F32)
    assert f1 > 0 and f1 % 256 == 0
    bad = [(0, 1, 1, 1, 16, 0, -1), (1, 1, 1, 1, 5, 0, -2), (1, 1, 1, 1, 16, 7, -2), (70000, 1, 1, 1, 16, 0, -2)]
    for B, H, N, M, d, dt, want in bad:
        shp = binding.FlareShape(B, H, N, M, d, dt)
        assert lib.flare_workspace_bytes(ctypes.byref(shp), None, None) == want
    assert lib.flare_workspace_bytes(None, None, None) == -1
    shp = binding.FlareShape(1, 1, 8, 32, 16, binding.FLARE_F32, 0, 2)      # shared_latents must be 0 or 1
    assert lib.flare_workspace_bytes(ctypes.byref(shp), None, None) == -1
    shp = binding.FlareShape(1, 1, 8, 32, 16, binding.FLARE_F32, 0, 0, 0, 4)   # unknown variant bit
    assert lib.flare_workspace_bytes(ctypes.byref(shp), None, None) == -1
    shp = binding.FlareShape(1, 1, 8, 32, 16, binding.FLARE_F32, 0, 0, 0, 3)   # both known bits
    assert lib.flare_workspace_bytes(ctypes.byref(shp), None, None) == 0


def test_null_and_misaligned_pointers_are_rejected(lib):
    shp = binding.FlareShape(1, 1, 8, 32, 16, binding.FLARE_F32)
    p = ctypes.c_void_p(4096)        # never dereferenced: the checks fail first
    odd = ctypes.c_void_p(4100)
    one = ctypes.c_float(1)
    assert lib.flare_forward(ctypes.byref(shp), None, p, p, p, p, p, None, one, p, 1 << 20, None) == -1
    assert lib.flare_forward(ctypes.byref(shp), p, p, p, None, p, p, None, one, p, 1 << 20, None) == -1
    assert lib.flare_forward(ctypes.byref(shp), p, odd, p, p, p, p, None, one, p, 1 << 20, None) == -3
    assert lib.flare_forward(ctypes.byref(shp), p, p, p, p, p, p, odd, one, p, 1 << 20, None) == -3
    assert lib.flare_forward(ctypes.byref(shp), p, p, p, p, p, p, None, one, p, 16, None) == -4
    assert lib.flare_forward(ctypes.byref(shp), p, p, p, p, p, p, None, one, None, 0, None) == -4
    assert lib.flare_decode(ctypes.byref(shp), p, p, None, p, None, one, None, 0, None) == -1
    # the entry point with the static scratch: shape and size checks come before anything touches a device
    big = binding.FlareShape(1, 8, 1 << 20, 2048, 8, binding.FLARE_BF16)
    assert lib.flare_forward_static(ctypes.byref(big), p, p, p, p, p, p, None, one, None) == -6
    assert lib.flare_forward_static(None, p, p, p, p, p, p, None, one, None) == -1
    assert lib.flare_backward(ctypes.byref(shp), p, p, p, None, None, None, p, p, p, p, p, one, p,
                              1 << 20, None) == -1
    assert lib.flare_backward(ctypes.byref(shp), p, p, p, None, None, p, p, p, p, p, p, one, p,
                              16, None) == -4


def test_native_half_loads_by_itself(lib):
    """The native half of the binding loads in a program that has not imported torch yet."""
    import subprocess
    import sys
    code = "from paper_2508_12594_amd import binding; print(binding._native().__name__)"
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("_native"), r.stderr
