"""Registers and private memory of kernels whose speed hangs on them, from the
compiler's resource report of the build's own flags (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_18052_amd import build


def _report(source):
    """{kernel or function: {"VGPRs": n, "ScratchSize": bytes a lane}}"""
    if not (shutil.which(build.HIPCC) or os.path.exists(build.HIPCC)):
        pytest.skip("no hipcc")
    cmd = [build.HIPCC, "-x", "hip"] + build.COMMON + build.EXTRA.get(source, []) + [
        "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(build.CSRC, source), "-o",
        os.devnull]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    out, cur = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
        m = re.search(r"remark: .*?\s(VGPRs|ScratchSize)(?: \[bytes/lane\])?: (\d+)", line)
        if m and cur is not None:
            cur[m.group(1)] = int(m.group(2))
    return out


def _kernel(report, name):
    found = [v for k, v in report.items() if name in k]
    assert len(found) == 1, sorted(report)
    return found[0]


def test_vote_keeps_its_matrix_in_registers():
    """The cubic of a full-rank matrix is a function of its own; its nine
    entries go to it in registers."""
    assert _kernel(_report("fea_focal.hip"), "k_fv_vote")["ScratchSize"] == 0


def test_per_match_camera_kernel_keeps_three_waves_per_simd():
    """512 registers per SIMD lane in blocks of 8: at most 168 for a third
    wave, without which 3,000 cameras take a second round."""
    r = _kernel(_report("fea_camera.hip"), "k_camgradILb0")
    assert r["VGPRs"] <= 168 and r["ScratchSize"] == 0
