"""What the compiler made of kernels whose speed rests on their registers, read from the metadata in the built library.  No
GPU needed."""
import os
import re
import struct

import msgpack
import pytest

from paper_2508_12594_amd import binding


@pytest.fixture(scope="module")
def kernels():
    """Metadata of every kernel in libflare.so, by mangled name."""
    if not os.path.exists(binding.LIB_PATH):
        from paper_2508_12594_amd import build
        build.build_library(verbose=False)
    with open(binding.LIB_PATH, "rb") as f:
        blob = f.read()
    found, at = {}, 0
    while True:
        at = blob.find(b"\x7fELF\x02\x01", at + 1)
        if at < 0:
            break
        if struct.unpack_from("<H", blob, at + 18)[0] != 224:    # EM_AMDGPU
            continue
        shoff = struct.unpack_from("<Q", blob, at + 40)[0]
        shentsize, shnum = struct.unpack_from("<HH", blob, at + 58)
        for i in range(shnum):
            kind, _, _, off, size = struct.unpack_from("<IQQQQ", blob, at + shoff + i * shentsize + 4)
            if kind != 7:                                        # SHT_NOTE
                continue
            p, end = at + off, at + off + size
            while p < end:
                nsz, dsz, ntype = struct.unpack_from("<III", blob, p)
                name, desc = p + 12, p + 12 + (nsz + 3) // 4 * 4
                if blob[name:name + 6] == b"AMDGPU" and ntype == 32:
                    for k in msgpack.unpackb(blob[desc:desc + dsz], raw=False)["amdhsa.kernels"]:
                        found[k[".name"]] = k
                p = desc + (dsz + 3) // 4 * 4
    return found


def spilled(kernels, head, latent_tiles):
    pat = re.compile(r"bwd_dkdv_planned_kernelILi%dELi%dELb1E" % (head, latent_tiles))    # (the form that also makes dQ)
    counts = [k[".vgpr_spill_count"] for n, k in kernels.items() if pat.search(n)]
    assert len(counts) >= 2, "no such kernels in the library"
    return max(counts)


@pytest.mark.parametrize("latent_tiles,most", [(1, 0), (2, 0), (3, 0), (4, 0), (5, 0), (6, 0), (7, 11), (8, 27)])
def test_dkdv_registers_at_16_columns(kernels, latent_tiles, most):
    """Seven and eight latent tiles have never fitted with two exponentials; up to six fit."""
    assert spilled(kernels, 16, latent_tiles) <= most


@pytest.mark.parametrize("head,latent_tiles,most", [(4, 1, 0), (4, 2, 0), (4, 4, 0), (4, 8, 5)] + [(8, t, 0) for t in range(1, 7)] +
                         [(8, 7, 2), (8, 8, 9)])
def test_dkdv_registers_at_4_and_8_columns(kernels, head, latent_tiles, most):
    assert spilled(kernels, head, latent_tiles) <= most


@pytest.mark.parametrize("latent_tiles", [1, 2, 3, 4, 6, 8])
def test_dkdv_registers_at_32_columns(kernels, latent_tiles):
    """With two exponentials every value spilled is written and read again in each token tile: 26 to 39 of them made the
    kernel take half as long again (a few that are read once a tile do not show)."""
    assert spilled(kernels, 32, latent_tiles) <= 4


@pytest.mark.parametrize("latent_tiles,waves", [(1, 4), (2, 3)])
def test_wide_head_decode_keeps_its_waves(kernels, latent_tiles, waves):
    """The launch counts on so many workgroups of four waves on a CU (512 registers a lane and SIMD, given in eights)."""
    pat = re.compile(r"decode_mfma_kernelILi32ELi%dELb1E" % latent_tiles)
    counts = {n: k[".vgpr_count"] for n, k in kernels.items() if pat.search(n)}
    assert len(counts) >= 6, "no such kernels in the library"      # (two storage types, merging or not, token statistics)
    assert all(-(-c // 8) * 8 * waves <= 512 for c in counts.values()), counts


@pytest.mark.parametrize("head", [4, 8, 16])
@pytest.mark.parametrize("form", [1, 2])
def test_fp32_kernel_that_forms_dq_too_spills_nothing(kernels, head, form):
    """dQ of four latent tiles lies in registers beside everything else (253 of 256 at 16 columns), two waves to a SIMD; a value
    spilled would be written and read again in every token tile."""
    pat = re.compile(r"token_pass_f32_kernelILi%dELi2ELi1ELb[01]ELi%dE" % (head, form))
    found = {n: (k[".vgpr_spill_count"], k[".vgpr_count"]) for n, k in kernels.items() if pat.search(n)}
    assert len(found) == 2, "no such kernels in the library"         # (merging dZ or not)
    assert all(spills == 0 and count <= 256 for spills, count in found.values()), found


def test_arguments_of_the_fp32_token_kernels_in_four_lines(kernels):
    """Short forwards wait for every 64-byte line of arguments; what a kernel reads behind its own is the workgroup's size."""
    ends = {}
    for n, k in kernels.items():
        if "token_pass_f32_kernel" in n:
            used = [a for a in k[".args"] if not a[".value_kind"].startswith("hidden_") or "block_count" in a[".value_kind"] or
                    "group_size" in a[".value_kind"]]
            ends[n] = max(a[".offset"] + a[".size"] for a in used)
    assert len(ends) >= 40, "no such kernels in the library"
    assert max(ends.values()) <= 256, ends
