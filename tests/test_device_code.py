"""CPU checks of the gfx950 code that the build puts into libtlf.so."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_15160_amd import build, tlf

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def disassembly(tmp_path_factory):
    """Disassembled instruction lines of every source's device code, in order."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(tlf.LIB_PATH):
        build.build()
    d = tmp_path_factory.mktemp("device_code")
    lib = shutil.copy(tlf.LIB_PATH, d)  # the bundles are extracted beside the library
    subprocess.check_call([OBJDUMP, "--offloading", lib], cwd=d, stdout=subprocess.DEVNULL)
    lines = []
    for name in sorted(os.listdir(d)):
        if name.endswith("gfx950"):
            lines += subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", str(d / name)], text=True).splitlines()
    return lines


def test_lds_loads_keep_a_wait_state_from_m0(disassembly):
    """A scalar write of M0 must be one wait state ahead of a load from global
    memory into LDS, which takes its LDS address from it."""
    loads, close = 0, []
    before = ""
    for line in disassembly:
        m = re.match(r"\s+([a-z]\w+)\s*([^/]*)", line)
        if not m:
            continue
        if re.match(r"(global|buffer|scratch)_load_lds_", m[1]):
            loads += 1
            if re.match(r"s_\w+ m0\b", before):
                close.append(line.strip())
        before = f"{m[1]} {m[2]}"
    assert loads > 0
    assert not close, f"{len(close)} of {loads} loads into LDS follow a write of M0 directly"
