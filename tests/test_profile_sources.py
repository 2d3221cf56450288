"""The revision that stored counters carry changes with every source file that the sweep kernel is compiled from."""
import os
import re
import shutil

from conftest import ROOT
from paper_2605_06046_amd.profile_summary import kernel_rev

CSRC = os.path.join("paper_2605_06046_amd", "csrc")


def test_every_source_of_the_sweep_counts(tmp_path):
    shutil.copytree(os.path.join(ROOT, CSRC), tmp_path / CSRC)
    rev = kernel_rev(str(tmp_path))
    assert rev == kernel_rev(ROOT)
    todo, files = ["fea_sweep_mfma.hip"], set()
    while todo:
        name = todo.pop()
        if name not in files:
            files.add(name)
            todo += re.findall(r'#include "(fea_[^"]+)"', (tmp_path / CSRC / name).read_text())
    assert {"fea_sweep_mfma.hip", "fea_sweep_core.inc", "fea_plan.h", "fea_tile.h"} <= files
    for name in sorted(files):
        path = tmp_path / CSRC / name
        text = path.read_text()
        path.write_text(text + "\n")
        assert kernel_rev(str(tmp_path)) != rev, name
        path.write_text(text)
    with open(tmp_path / CSRC / "fea_append.hip", "a") as f:
        f.write("\n")
    assert kernel_rev(str(tmp_path)) == rev
