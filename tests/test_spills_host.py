"""The kernels whose register count is planned by hand (rows or accumulator tiles
held in registers) compile without spills or scratch: a spilled register of the
loss-only kernel is a scratch store and load per lane of every row (no GPU
needed; skipped when hipcc is absent)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_17826_amd import build_lib as B

HIPCC = B.HIPCC if os.path.exists(B.HIPCC) else shutil.which("hipcc")
pytestmark = pytest.mark.skipif(not HIPCC, reason="hipcc not available")

_KERNEL = re.compile(r"\.name:\s+(\S+).*?\.private_segment_fixed_size:\s+(\d+).*?"
                     r"\.sgpr_spill_count:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)", re.S)


@pytest.mark.parametrize("src", ["k_logits.hip", "k_gemm_mfma.hip", "k_gemm_f32.hip"])
def test_no_spills(src, tmp_path):
    out = tmp_path / (src + ".s")
    cmd = [HIPCC, *[f for f in B.CFLAGS if f != "-fPIC"], *B.SOURCE_FLAGS.get(src, []),
           "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = _KERNEL.findall(out.read_text())
    assert kernels
    bad = [k for k in kernels if any(int(x) for x in k[1:])]
    assert not bad, bad
