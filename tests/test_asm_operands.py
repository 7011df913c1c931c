"""Register operands of the on-chip solve's multiply-add chains.

A chain writes its two sums with its first instructions and reads its other
inputs in later ones, so neither sum may share a register with an input, also
where the compiler knows the two to hold the same value at the start.  The
assembly of the kernels, and of probes whose sums start as such a value, is
searched for a chain that does.
"""
import os
import re
import subprocess

import pytest

from paper_2309_06427_amd import build_lib

PROBE = """
#include "{src}"
namespace ssp {{
__global__ void probe(const float *in, float *out) {{
    const float z = in[0];
    float a[14], s0 = z, s1 = z, t0 = 0.0f, t1 = 0.0f, c[14];
    for (int j = 0; j < 14; ++j) a[j] = z, c[j] = 0.0f;
    chain13<0>(a, z, s0, s1);
    chain13<1>(c, z, t0, t1);
    out[threadIdx.x] = s0 + s1 + t0 + t1;
    s0 = s1 = z, t0 = t1 = 0.0f;
    chain14(a, z, s0, s1);
    chain14(c, z, t0, t1);
    out[threadIdx.x + 64] = s0 + s1 + t0 + t1;
    s0 = s1 = z, t0 = t1 = 0.0f;
    chain6(a, z, s0, s1);
    chain6(c, z, t0, t1);
    out[threadIdx.x + 128] = s0 + s1 + t0 + t1;
}}
}}
"""


def test_chain_sums_share_no_register_with_their_inputs(tmp_path):
    try:
        cc = build_lib.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE.format(src=os.path.join(build_lib.CSRC, "pcg4.hip")))
    subprocess.run([cc, *build_lib.flags(), "-S", "--cuda-device-only", str(src), "-o", str(out)], check=True,
                   capture_output=True)
    chains = re.findall(r"ASMSTART(.*?)ASMEND", out.read_text(), flags=re.S)
    seen = 0
    for c in chains:
        ops = re.findall(r"v_fmac_f32_dpp (v\d+), (v\d+), (v\d+) ", c)
        if not ops:
            continue
        seen += 1
        sums = {o[0] for o in ops}
        assert len(sums) == 2, c
        assert not sums & ({o[1] for o in ops} | {o[2] for o in ops}), c
    assert seen > 12  # the probes' six and the kernels'
