"""Tile shapes of the stage kernel: the x and y reconstructions take two cells at a time, so
a build with an odd tile is refused by the compiler (CPU only, front end of hipcc)."""
import os
import subprocess

import pytest

from paper_2402_05193_amd import build as B


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("bx,by,ok", [(32, 8, True), (15, 16, False), (16, 9, False)])
def test_tile_shape(bx, by, ok):
    r = subprocess.run([B.HIPCC, *B.FLAGS, "-fsyntax-only", f"-DTILE_BX={bx}", f"-DTILE_BY={by}", "-DTILE_NT=320",
                        "-DFV_REAL=float", "-DFV_MODEL=EULER", "-DFV_REC=0", os.path.join(B.CSRC, "fv_stage_inst.hip")],
                       capture_output=True, text=True, timeout=300)
    assert (r.returncode == 0) == ok, r.stderr[-2000:]
    assert ok or "two cells at a time" in r.stderr
