"""The inline-asm blocks of the circuit kernels, compiled for gfx950 with operands the compiler knows to
hold equal values: no register that a block writes may also hold another operand it still reads."""
import os
import re
import subprocess

import pytest

from paper_2506_23246_amd import build as B

PROBE = """
#include "%s/fused_kernel.hpp"
namespace qp {
// amplitudes known to be zero, as the sums start from
__global__ void k_stat(const float* in, float* out) {
  float sr[8][8], si[8][8];
  for (int r = 0; r < 8; ++r) {
    sr[0][r] = 0.f; si[0][r] = 0.f;
    sr[4][r] = in[threadIdx.x * 16 + r]; si[4][r] = in[threadIdx.x * 16 + 8 + r];
  }
  float sx = 0.f, sy = 0.f;
  stat_lane<K, 0>(sr, si, sx, sy);
  out[threadIdx.x * 2] = sx; out[threadIdx.x * 2 + 1] = sy;
}
// an amplitude known to equal the tangent
__global__ void k_rot(const float* in, float* out) {
  float sr[8][8], si[8][8];
  const float t = in[threadIdx.x];
  for (int r = 0; r < 8; ++r) {
    sr[0][r] = r == 3 ? t : in[64 + threadIdx.x * 16 + r]; si[0][r] = in[64 + threadIdx.x * 16 + 8 + r];
  }
  rot_lane<K, 0>(sr, si, t);
  for (int r = 0; r < 8; ++r) { out[threadIdx.x * 16 + r] = sr[0][r]; out[threadIdx.x * 16 + 8 + r] = si[0][r]; }
}
}
"""


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="no hipcc")
@pytest.mark.parametrize("K", range(4))
def test_outputs_have_registers_of_their_own(K, tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text((PROBE % B.CSRC).replace("<K, 0>", f"<{K}, 0>"))
    asm = tmp_path / "probe.s"
    subprocess.run([B.HIPCC, *B.HIP_FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True,
                   capture_output=True, timeout=300)
    blocks = re.findall(r"#ASMSTART\n(.*?)#ASMEND", asm.read_text(), re.S)
    lanes = [b for b in blocks if "v_fmac_f32_dpp" in b]
    assert len(lanes) == 3      # two halves of the sums, one rotation
    for b in lanes:
        ops = [(d, x.lstrip("-"), y) for d, x, y in re.findall(r"v_fmac_f32_dpp (v\d+), (-?v\d+), (v\d+) ", b)]
        assert len(ops) == 16
        written = {d for d, _, _ in ops}
        for d, x, y in ops:
            assert y not in written and (x not in written or x == d and len(written) == 16), (d, x, y)
