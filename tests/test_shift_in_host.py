"""shift_in's carry-in comes from a scalar instruction whatever its arguments
are, in the assembly of a kernel that passes it compares and constants (no GPU):
a vector instruction that reads a mask right behind the compare that wrote it
would read the old one."""
import re
import subprocess

import pytest

from paper_2204_03756_amd import build as B

KERNEL = """
#include "mtpt_device.h"
using namespace mtpt;
__global__ void probe(const float* x, float lim, uint32_t* out)
{
    uint64_t in;
    uint32_t w = out[threadIdx.x];
    w = shift_in(w, __builtin_amdgcn_fcmpf(x[threadIdx.x], lim, kFcmpLe), %s, in);
    out[threadIdx.x] = w;
    out[threadIdx.x + 64] = __builtin_amdgcn_inverse_ballot_w64(in) ? 1u : 0u;
}
"""


@pytest.mark.parametrize("valid", ["~0ull", "__builtin_amdgcn_uicmp(w, 7u, kIcmpUlt)", "__builtin_amdgcn_ballot_w64(w > 3u)"])
def test_the_carry_is_a_scalar_result(tmp_path, valid):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(KERNEL % valid)
    subprocess.run([B.HIPCC, *B.FLAGS, "-I", B.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    body = text[text.index("probe", text.index("@_Z5probe")):text.index("s_endpgm")]
    lines = [l.strip() for l in body.split("\n") if re.match(r"\s*[sv]_", l)]
    at = [k for k, l in enumerate(lines) if l.startswith("v_addc_co_u32")]
    assert len(at) == 1, lines
    mask = lines[at[0]].split()[-1]
    writer = next(l for l in reversed(lines[:at[0]]) if len(l.split()) > 1 and l.split()[1].rstrip(",") == mask)
    assert writer.startswith("s_"), writer
