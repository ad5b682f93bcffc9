"""Loads straight to LDS take their place from m0, which the compiler uses too: it has to be told."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_compiler_itself_writes_m0_in_front_of_every_load(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path / "forms.s"
    done = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "--cuda-device-only", "-S", "-o", str(out),
                           os.path.join(HERE, "host", "load_to_lds_forms.hip")],
                          check=True, capture_output=True, text=True, timeout=600)
    # no register that the compiler reserves is changed behind its back
    assert "inline asm" not in done.stderr
    loads, place, own = 0, False, True
    for line in out.read_text().splitlines():
        line = line.strip()
        own = "#ASMEND" in line or (own and "#ASMSTART" not in line)
        if re.match(r"s_\w+ m0,", line):
            assert own, line
            place = True
        elif line.startswith("global_load_lds_"):
            assert place, line
            loads, place = loads + 1, False
    assert loads >= 8
