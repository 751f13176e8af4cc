"""Build-time switches reach every rule that depends on them: without the fused
N = 4096 kernels no rule may send a batch of that shape to them (the host side
would still report the fused path, for which there is then no detection kernel).
"""
import os
import shutil
import subprocess

import pytest

from paper_1411_3656_amd import build

SOURCE = """
#include "ppf_engine.h"
static_assert(ppf::fused_ok(4096, 8) == (PPF_FUSED_4096 != 0), "fused_ok");
static_assert(ppf::fused_by_long(4096, 8) == (PPF_FUSED_4096 != 0), "fused_by_long");
static_assert(ppf::fused_by_long(2048, 8) && !ppf::fused_by_long(1024, 8), "fused_by_long");
"""


@pytest.mark.parametrize("fused", [0, 1])
def test_fused_4096(tmp_path, fused):
    if not (os.path.exists("/opt/rocm/bin/hipcc") or shutil.which("hipcc")):
        pytest.skip("no hipcc")
    src = tmp_path / "switch.hip"
    src.write_text(SOURCE)
    res = subprocess.run([build.hipcc(), *build.COMMON, f"-DPPF_FUSED_4096={fused}", "-x", "hip", "--offload-device-only",
                          "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
