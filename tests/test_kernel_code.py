"""What the compiler makes of single device functions: the assembly of a small kernel around them.  No GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2508_12594_amd import build

SPLIT = """
#include "flare_mfma_common.h"
__global__ void split(const uint32_t *w, flare::HiLo *out, float c)
{
    out[threadIdx.x] = flare::split_scaled<%s>(w[threadIdx.x], c);
}
"""


def assembly(tmp_path, source):
    src, out = str(tmp_path / "k.hip"), str(tmp_path / "k.s")
    with open(src, "w") as f:
        f.write(source)
    subprocess.run(["hipcc"] + build.FLAGS + build.SOURCES["flare_mfma_bwd.hip"] +
                   ["-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only", "-S", "-o", out, src],
                   check=True, stderr=subprocess.DEVNULL)
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("f16", ["false", "true"])
def test_scaled_queries_are_split_as_rounded(tmp_path, f16):
    """The lo word is what the rounding of the fp32 product left: two products of their own, none inside a multiply-add."""
    code = assembly(tmp_path, SPLIT % f16)
    assert len(re.findall(r"\bv_(?:pk_)?mul_f32", code)) == 2
    fused = re.findall(r"\bv_(?:fma|fmac|mad|mac)\w*.*", code)
    # (fp16: the hi part may be widened within the subtraction, as a factor of 1)
    assert not [f for f in fused if not (f16 == "true" and "mix_f32" in f and re.search(r"\b1\.0\b", f))], fused
