"""The dispatch kernels keep everything in registers and LDS.

revive_dispatch_static is for callers that cannot allocate; a kernel with private scratch makes the runtime allocate
its backing memory when it is first launched.  The compiler's own report names the bytes per lane."""
import os
import re
import subprocess

import pytest

from paper_2602_21140_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_dispatch_kernels_use_no_private_scratch(tmp_path):
    cmd = [HIPCC, *build.HIPCC_FLAGS, "--offload-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(build.CSRC, "dispatch.hip"), "-o", str(tmp_path / "dispatch.o")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert len(names) == len(scratch) and any("dispatch_small_kernel" in n for n in names)
    assert not {n: s for n, s in zip(names, scratch) if s}
