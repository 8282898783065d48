"""What the compiler gives the kernels: none of them may use scratch memory (a
copy of an argument struct or a spilled register there costs every launch).
Cross-compiled with the build's own flags; no GPU is used."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from paper_2607_20211_amd import build


@pytest.mark.parametrize("source", [s for s in build.SOURCES if s not in ("drsf_api.hip", "drsf_server.hip")])
def test_no_kernel_uses_scratch(source, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("hipcc not available")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([hipcc, *flags, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, source), "-o", str(tmp_path / "x.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert names and len(names) == len(scratch)
    assert not [(n, s) for n, s in zip(names, scratch) if s], source
