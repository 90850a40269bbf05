"""No kernel keeps registers in scratch memory: what the compiler reports for each of them, compiled as
the library is. A retrieval build with 108 spilled registers gave wrong pairs now and then."""

from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2607_21848_amd import build as B


@pytest.mark.parametrize("source", [s for s in B.SOURCES if s.endswith(".hip")])
def test_no_scratch(source, tmp_path):
    try:
        cc = B.hipcc()
    except RuntimeError as e:
        pytest.skip(str(e))
    out = subprocess.run([cc, *B.compile_flags(), "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
                          os.path.join(B.CSRC, source), "-o", str(tmp_path / "device.o")], check=True, capture_output=True, text=True).stderr
    kernels = re.findall(r"Function Name: (\S+)", out)
    assert kernels and len(kernels) == len(set(kernels))
    for what in (r"ScratchSize \[bytes/lane\]", "SGPRs Spill", "VGPRs Spill"):
        figures = [int(x) for x in re.findall(what + r": (\d+)", out)]
        assert len(figures) == len(kernels) and not any(figures), list(zip(kernels, figures))
