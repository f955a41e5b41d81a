"""The sources compile without warnings (hipcc cross-compiles for the GPU on any host).

The compiler warns, among other things, where inline assembly names a register as clobbered that
it may hold a value in all the same: such code has no defined behaviour.
"""

import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2607_20739_amd import build as B


def _compile(src):
    cmd = [B.hipcc()] + B.common_flags() + ["--cuda-device-only", "-c", os.path.join(B.CSRC, src), "-o", os.devnull]
    return src, subprocess.run(cmd, capture_output=True, text=True, timeout=300)


def test_device_code_compiles_without_warnings():
    try:
        B.hipcc()
    except RuntimeError as e:
        pytest.skip(str(e))
    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as pool:
        for src, res in pool.map(_compile, [s for s in B.SOURCES if s.endswith(".hip")]):
            assert res.returncode == 0, (src, res.stderr[-2000:])
            assert B.warnings(res.stderr) == [], src


def test_warnings_are_found_in_the_compilers_output():
    text = "\n".join(["'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)",
                      "a.hip:3:1: warning: unused function 'f' [-Wunused-function]", "    3 | void f();",
                      "1 warning generated when compiling for gfx950."])
    assert B.warnings(text) == ["a.hip:3:1: warning: unused function 'f' [-Wunused-function]"]
    assert B.warnings("") == []


def test_inline_assembly_that_loads_registers_waits_for_them():
    """The compiler takes the results of an assembly block as there when it ends: one that reads
    memory into registers waits for it inside (loads that go to LDS have no results)."""
    blocks = 0
    for name in os.listdir(B.CSRC):
        with open(os.path.join(B.CSRC, name)) as f:
            text = f.read()
        for block in re.findall(r"asm\s+volatile\s*\((.*?)\);", text, re.S):
            if re.search(r"\b(ds_read|global_load_dword|buffer_load|s_load)", block):
                blocks += 1
                assert "s_waitcnt" in block, (name, block[:120])
    assert blocks >= 2
