"""Which launch shapes every model and precision takes: the same as ever, whatever the step
loop keeps in LDS (tuning files hold such shapes).  No GPU needed."""
from __future__ import annotations

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = """
from paper_1409_4923_amd import bmotor as B
for noise in range(32):
    for prec in (B.BM_F64, B.BM_F32):
        for ppl in (1, 2):
            for block in (64, 128, 256, 512):
                try:
                    B.bm_tune_set_default(1, 0, noise, prec, B.make_tune(ppl, block))
                    ok = 1
                except B.BMError as e:
                    assert e.code == B.BM_ERR_UNSUPPORTED
                    ok = 0
                print(noise, prec, ppl, block, ok)
"""


def test_accepted_shapes():
    # a process of its own: an installed shape stays installed
    out = subprocess.run([sys.executable, "-c", SRC], cwd=ROOT, capture_output=True, text=True, check=True).stdout
    rows = [tuple(map(int, line.split())) for line in out.split("\n") if line]
    assert len(rows) == 32 * 2 * 2 * 4
    for noise, prec, ppl, block, ok in rows:
        f32 = prec == 1
        jump_grid, kicks, flips = noise & 16, noise & 2, noise & 4
        lane = (160 if f32 else 192) if jump_grid else (96 if f32 else 192) if kicks else 0
        lane += 48 if flips else 0
        assert ok == (lane * ppl * block <= 65536 and (f32 or ppl == 1)), (noise, prec, ppl, block)
