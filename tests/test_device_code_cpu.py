"""Checks of the compiled gfx950 code (no GPU): what the assembler accepts but the hardware does not order."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2505_15781_amd", "libdkv.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def device_code(tmp_path_factory):
    """Instruction lines of every device code object of the library."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(LIB):
        from paper_2505_15781_amd.build import build
        build()
    d = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    objects = sorted(f for f in os.listdir(d) if f.endswith("gfx950"))
    assert objects
    return [subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=d, check=True, capture_output=True,
                           text=True).stdout.splitlines() for f in objects]


def test_no_load_to_lds_directly_behind_a_write_of_m0(device_code):
    """A load to LDS takes its LDS address from M0 and needs one wait state behind the scalar write of M0; without it the
    old address may be used. The compiler keeps that distance in its own code, not inside inline assembly."""
    loads = 0
    for lines in device_code:
        for before, line in zip(lines, lines[1:]):
            if re.search(r"\b(global|buffer|scratch)_load_lds_|\b(global|buffer)_load_\w+ .*\blds\b", line):
                loads += 1
                assert not re.match(r"\s*s_\w+ m0\b", before), (before.strip(), line.strip())
    assert loads > 1000            # the tile kernels are made of them
