"""Registers of the adjoint kernels that add with device atomics (host only).

They hide the atomics behind other wavefronts: 512 registers per SIMD lane in
steps of 8 leave five of them up to 96 registers, four beyond (FP64 points at
1.5 m, 72,900 of them: 31 us with five, 35 with four)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_26222_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_five_wavefronts_per_simd(tmp_path):
    out = tmp_path / "eval.s"
    cmd = [build.HIPCC, *build.COMMON, "--cuda-device-only", "-S",
           os.path.join(build.CSRC, "eval.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    # k_eval_adjoint<T, POSE, PLANES = false, 0>
    got = dict(re.findall(r"\.amdhsa_kernel (\S*k_eval_adjointI[df]Lb[01]ELb0ELi0E\S*)"
                          r"[\s\S]*?\.amdhsa_next_free_vgpr (\d+)", out.read_text()))
    assert len(got) == 4
    assert max(int(v) for v in got.values()) <= 96, got
