"""The multi-instruction blocks of inline assembly write their result before they have
read every input, so no input may share a register with it.  Compiled for the GPU here
(nothing runs), with inputs of the result's own value, which the compiler would put in
one register."""
import os
import re
import subprocess

import pytest

from paper_2404_04994_amd import build as B

PROBE = r"""
#include "qa_internal.h"
__global__ void k_dot(const double *p, double *o)
{
    const double a = p[threadIdx.x], x = p[64 + threadIdx.x];
    double t[16];
    for (int q = 0; q < 16; ++q) t[q] = q < 6 ? a : p[128 + 64 * q + threadIdx.x];
    o[threadIdx.x] = qa::row_dot16(a, x, t);
}
__global__ void k_axpy(const double *p, double *o)
{
    const double f = p[threadIdx.x];
    double r[8];
    for (int q = 0; q < 8; ++q) r[q] = q & 1 ? f : p[64 * q + threadIdx.x];
    qa::row_axpy8<3>(r, f);
    for (int q = 0; q < 8; ++q) o[64 * q + threadIdx.x] = r[q];
}
"""


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="no hipcc")
def test_inputs_keep_their_registers(tmp_path):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    subprocess.check_call([B.HIPCC, *B.FLAGS, "-I", os.path.join(B.HERE, "csrc"),
                           "--cuda-device-only", "-S", "-o", str(out), str(src)],
                          stderr=subprocess.DEVNULL)
    blocks = re.findall(r"#ASMSTART(.*?)#ASMEND", out.read_text(), re.S)
    blocks = [re.findall(r"v_fmac_f64_dpp (\S+), (\S+), (\S+) row_newbcast", b) for b in blocks]
    blocks = [b for b in blocks if b]
    assert sorted(len(b) for b in blocks) == [8, 16]
    for b in blocks:
        written = {dst for dst, _, _ in b}
        assert not written & {factor for _, _, factor in b}
        for dst, lane_operand, _ in b:
            assert lane_operand == dst or lane_operand not in written
