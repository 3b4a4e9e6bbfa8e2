"""Reading the surrogate's parameters, gradient and loss, any of them, with
memory for one copy of everything and without: no exception leaves the call."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_read_with_and_without_host_memory(tmp_path):
    exe = str(tmp_path / "mlp_read")
    subprocess.run(["hipcc", "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1",
                    "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2002_03120_amd", "csrc"),
                    os.path.join(ROOT, "tests", "mlp_read_main.hip"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    assert len(out.splitlines()) == 32 and "wrong" not in out
