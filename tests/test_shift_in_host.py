"""shift_in's carry-ins come from scalar instructions whatever its arguments
are, in the assembly of kernels that pass it compares and constants (no GPU): a
vector instruction that reads a mask right behind the compare that wrote it
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
    constexpr int U = %d;
    uint32_t w = out[threadIdx.x];
    uint64_t near[U], valid[U], in[U];
    for (int u = 0; u < U; ++u) {
        near[u] = __builtin_amdgcn_fcmpf(x[threadIdx.x + 64 * u], lim, kFcmpLe);
        valid[u] = %s;
    }
    w = shift_in(w, near, valid, in);
    out[threadIdx.x] = w;
    for (int u = 0; u < U; ++u)
        out[threadIdx.x + 64 * (u + 1)] = __builtin_amdgcn_inverse_ballot_w64(in[u]) ? 1u : 0u;
}
"""


@pytest.mark.parametrize("valid", ["~0ull", "__builtin_amdgcn_uicmp(w + u, 7u, kIcmpUlt)"])
@pytest.mark.parametrize("width", [1, 2, 4])
def test_the_carries_are_scalar_results(tmp_path, width, valid):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(KERNEL % (width, valid))
    subprocess.run([B.HIPCC, *B.FLAGS, "-I", B.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    body = text[text.index("@_Z5probe"):text.index("s_endpgm")]
    lines = [l.strip() for l in body.split("\n") if re.match(r"\s*[sv]_", l)]
    at = [k for k, l in enumerate(lines) if l.startswith("v_addc_co_u32")]
    assert len(at) == width, lines
    for k in at:
        mask = lines[k].split()[-1]
        writer = next(l for l in reversed(lines[:k]) if len(l.split()) > 1 and l.split()[1].rstrip(",") == mask)
        assert writer.startswith("s_and_b64"), writer
