"""Vector registers of the hot kernels, as the compiler reports them for the package's own flags (no GPU).

A register that spills to scratch memory inside these kernels costs a round trip per lane in their inner loops, and
no result shows it.
"""
import os
import re
import subprocess

import pytest

from paper_2211_12858_amd import build as sb_build


def spilled_registers(source, tmp_path):
    """Kernel name with its template arguments -> spilled vector registers."""
    try:
        cc = sb_build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc is not available")
    flags = [f for f in sb_build.HIPCC_FLAGS if f != "-shared"]
    res = subprocess.run([cc] + flags + ["-Rpass-analysis=kernel-resource-usage", "--offload-device-only", "-c", "-o",
                                         str(tmp_path / "kernels.o"), os.path.join(sb_build.CSRC, source)],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-2000:]
    out, name = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"remark: +VGPRs Spill: (\d+)", line)
        if m:
            out[name] = int(m.group(1))
    names = subprocess.run(["c++filt"] + list(out), capture_output=True, text=True).stdout.splitlines()
    return {re.sub(r"\(anonymous namespace\)::|sb::|void ", "", n).split("(")[0]: v for n, v in zip(names, out.values())}


@pytest.mark.parametrize("source,kernel,instances", [("sb_hist.hip", "k_hist_rot<", 5),
                                                      ("sb_sketch.hip", "k_project_mfma4<", 13)])
def test_no_spilled_registers(source, kernel, instances, tmp_path):
    spilled = {n: v for n, v in spilled_registers(source, tmp_path).items() if n.startswith(kernel)}
    assert len(spilled) == instances
    assert all(v == 0 for v in spilled.values()), spilled
