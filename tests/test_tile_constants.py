"""The pass kernel's tuning constants: a value its loops cannot run with does not compile."""

import os
import subprocess

import pytest

from paper_2309_04255_amd import build


def _check(*defines):
    """Device-side syntax check of the pass kernel: (return code, compiler output)."""
    cmd = [build.hipcc(), *build.compile_flags(), "-fsyntax-only", "--cuda-device-only", *defines,
           os.path.join(build.CSRC, "pass.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    return r.returncode, r.stdout + r.stderr


# A row-split tile shares each k-step's weights two steps ahead, from a stage
# that an earlier step has refilled: that takes four register stages or more
# (two would share the previous weights again), and an even number of them.
@pytest.mark.parametrize("define", ["-DLLMCAD_ROW_DEPTH=2", "-DLLMCAD_ROW_DEPTH=3", "-DLLMCAD_STAGE_REGS=12"])
def test_row_tile_depth_is_refused(define):
    rc, out = _check(define)
    assert rc != 0 and "shares weights two k-steps ahead" in out


@pytest.mark.parametrize("define", ["-DLLMCAD_ROW_DEPTH=4", "-DLLMCAD_ROW_DEPTH=7", "-DLLMCAD_ROW_DEPTH=8"])
def test_row_tile_depth_is_taken(define):
    rc, out = _check(define)
    assert rc == 0, out
