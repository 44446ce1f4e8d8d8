"""Host check of the group walk's cell numbering (sph_walk_cell.h) against integer
division, over every cell of boxes up to 512^3."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="needs hipcc")
def test_box_cell_is_integer_division(tmp_path):
    exe = str(tmp_path / "walk_cell_check")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-ffp-contract=off",
                    "-I", os.path.join(ROOT, "paper_2005_02656_amd", "csrc"),
                    os.path.join(HERE, "walk_cell_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    rows = [list(map(int, ln.split())) for ln in r.stdout.split("\n") if ln.strip()]
    assert len(rows) == 14, r.stdout + r.stderr
    for nx, ny, nz, wrong, outside in rows:
        assert wrong == 0 and outside == 0, (nx, ny, nz, wrong, outside)
    assert r.returncode == 0
