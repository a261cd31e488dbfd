"""The asm of the asynchronous copy declares that it writes m0, the register
that holds the LDS address of every such copy: a builtin copy after it must set
m0 again, also to an address that it had set before.  Compiled for gfx950, not
run."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_builtin_copies_after_the_asm_copy_set_m0_again(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path / "mix.s")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-S",
                        "--offload-device-only", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", os.path.join(HERE, "native", "async_copy_mix.hip"),
                        "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    code = open(out).read()
    body = code[code.index("async_copy_mix"):]
    events = re.findall(r"^\s*(?:s_mov\w*\s+(m0),|(global_load_lds_dwordx4)\s)", body, re.M)
    order = "".join("m" if m0 else "c" for m0, _ in events)
    assert order.count("c") == 3, order
    # a write of m0 before each of the three copies
    assert re.fullmatch(r"m+cm+cm+c", order), order
