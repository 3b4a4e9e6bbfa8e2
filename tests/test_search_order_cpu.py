"""The search visits the partners of a particle in the same order whether one
thread or several lanes walk its cells: the walks of the device header, run on
the host over boxes of 3 to 11 cells in x, walls, shear and reaches 1 to 3."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_one_thread_and_several_lanes_find_partners_in_the_same_order(tmp_path):
    exe = str(tmp_path / "search_order")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O2",
                    "-ffp-contract=off", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2002_03120_amd", "csrc"),
                    os.path.join(ROOT, "tests", "search_order_main.hip"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    rows = [[int(v) for v in line.split()] for line in out.splitlines()]
    assert len(rows) == 3 * 9 * 2 * 4
    differ = 0
    for *box, short, pruned32, pruned64, exact32, exact64, ordered in rows:
        # the lanes' kernels take the exact rows in boxes of a short axis
        assert exact32 == exact64 == 0, box
        assert ordered == 0, box
        if not short:
            assert pruned32 == pruned64 == 0, box
        differ += pruned32 + pruned64 > 0
    assert differ  # pruned rows alone would not do
