"""Listing check of DPP reads behind lane swaps (host only): v_permlane16_swap,
v_permlane32_swap and v_swap write both of their operands, so a DPP read needs
its two wait states behind either. The scanner is checked on a planted listing."""
import os
import shutil
import subprocess

import pytest

from paper_2509_26222_amd import build
from test_dpp_hazards import _vregs

SWAPS = ("v_permlane16_swap", "v_permlane32_swap", "v_swap")


def swap_hazards(listing):
    """(number of swaps, list of (swap, DPP reader of one of its operands))."""
    ins = [t for t in (line.strip() for line in listing.splitlines())
           if t and not t.startswith((";", ".")) and not t.endswith(":")]
    found, n = [], 0
    for i, t in enumerate(ins):
        if not t.startswith(SWAPS):
            continue
        n += 1
        a, b = (o.strip().split()[0] for o in t.split(None, 1)[1].split(",")[:2])
        dst = _vregs(a) | _vregs(b)
        waits = 0
        for u in ins[i + 1:]:
            if waits >= 2:
                break
            op = u.split()[0]
            if "_dpp" in op:
                src = u.split(None, 1)[1].split(",")[1].strip().split()[0].lstrip("-")
                if _vregs(src) & dst:
                    found.append((t, u))
                    break
            waits += int(u.split()[1]) + 1 if op == "s_nop" else 1
    return n, found


def test_scanner_finds_planted_swaps():
    listing = "\n".join([
        "\tv_permlane32_swap_b32_e32 v2, v5",
        "\tv_mov_b32_dpp v12, v5 row_newbcast:2 row_mask:0xf bank_mask:0xf",
        "\tv_permlane16_swap_b32_e32 v2, v5",
        "\tv_add_f64 v[10:11], v[0:1], v[0:1]",
        "\tv_fmac_f64_dpp v[6:7], v[2:3], v[8:9] row_newbcast:1 row_mask:0xf bank_mask:0xf",
        "\tv_swap_b32 v2, v5",
        "\ts_nop 1",
        "\tv_mov_b32_dpp v12, v2 row_newbcast:2 row_mask:0xf bank_mask:0xf",
    ])
    n, found = swap_hazards(listing)
    assert n == 3 and [f[0].split()[0] for f in found] == [
        "v_permlane32_swap_b32_e32", "v_permlane16_swap_b32_e32"]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_update_kernels_have_no_swap_hazard(tmp_path):
    out = tmp_path / "update.s"
    cmd = [build.HIPCC, *build.COMMON, "--cuda-device-only", "-S",
           os.path.join(build.CSRC, "update.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    n, found = swap_hazards(out.read_text())
    assert n > 100  # the factor's column exchanges
    assert not found, found[:5]
