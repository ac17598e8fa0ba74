"""Copies from global memory to LDS take their LDS address from M0 and their base from scalar registers.  The hardware needs
a wait state between an instruction that writes M0 and the copy, and five between a vector instruction that writes one of
those scalar registers and the copy.  The compiler keeps them between instructions of its own but does not look into
inline assembly, so the code in the built library is checked."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_21140_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
WRITES_M0 = re.compile(r"s_\w+ m0\b")
WRITES_SCALAR = re.compile(r"v_\w+ (?:s(\d+)|s\[(\d+):(\d+)\])")  # a vector instruction's scalar result
BASE = re.compile(r"global_load_lds_\w+ \S+ s\[(\d+):(\d+)\]")


def wait_states(text):
    return 1 + int(text.split()[1]) if text.startswith("s_nop") else 1


def late_base(history, copy):
    """The vector instruction that wrote the copy's base less than five wait states ahead of it, or none."""
    base, passed = BASE.match(copy), 0
    for text in reversed(history):
        if not base or passed >= 5:
            return None
        w = WRITES_SCALAR.match(text)
        if w and int(w[1] or w[2]) <= int(base[2]) and int(w[1] or w[3]) >= int(base[1]):
            return text
        passed += wait_states(text)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_wait_states_in_front_of_copies_to_lds(tmp_path):
    if not os.path.exists(build.LIB_PATH):
        build.build(verbose=False)
    lib = shutil.copy(build.LIB_PATH, tmp_path)  # the code objects are written beside the file
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    where, history, copies, bad = "", [], {}, []
    for obj in sorted(tmp_path.glob("*gfx950*")):
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(obj)], check=True, capture_output=True, text=True)
        for line in r.stdout.splitlines():
            text = line.split("//")[0].strip()
            if text.startswith("<") and text.endswith(">:"):
                where, history = text[1:-2], []
                continue
            if "global_load_lds" in text or (text.startswith("buffer_load") and text.endswith(" lds")):
                copies[where] = copies.get(where, 0) + 1
                if history and WRITES_M0.match(history[-1]):
                    bad.append((where, history[-1], text))
                late = late_base(history, text)
                if late:
                    bad.append((where, late, text))
            if text:
                history = history[-7:] + [text]
    for kernel in ("gemm_bf16_dma_kernel", "router_tile_kernel"):
        assert any(kernel in name for name in copies)
    assert not bad, (len(bad), bad[:3])
