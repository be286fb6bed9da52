"""The device header with inline assembly compiles without a word: its warning bracket encloses every statement that names a
reserved register and leaves the state of an including file as it was."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1904_08368_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_lds_dma_header_is_quiet_and_balanced(tmp_path):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    src = tmp_path / "use.hip"
    src.write_text('#include "lds_dma.hpp"\n'
                   "__global__ void k(relay::intx4 r) { relay::l2_touch(r, 0u, threadIdx.x); relay::lds_dma16(r, 0u, threadIdx.x); }\n")
    out = subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-device-only", "-std=c++17", "-I", CSRC, "-Wall", "-Wno-unused-command-line-argument", "-S", "-o", os.devnull, str(src)],
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    assert "warning" not in out.stderr, out.stderr
