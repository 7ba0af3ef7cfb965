"""Frames of every width modulo four, whose rows start and end off the four
pixels that a lane stores at once: each image bit for bit, its neighbours in
memory included, against the oracle.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda
from tests.gpu_util import compare_render

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (2, 3), (3, 2), (4, 1), (5, 5), (17, 16), (15, 33), (18, 17), (31, 31), (33, 8), (34, 9), (35, 10),
         (36, 11), (61, 67), (62, 5), (63, 64), (99, 3), (129, 18)]


# images one after the other in memory, so that each starts where the one before
# it ends; two-kernel and fused passes, tiles of every size, empty ones among them
@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("look", ["flat", "fused", "smooth"])
def test_rows_off_four_pixels(tile, look):
    oracle.lib()
    s = sg.make_scene(2100, [9] * len(SIZES), 32, mixed=True)
    s.cam_w[:] = [w for w, _ in SIZES]
    s.cam_h[:] = [h for _, h in SIZES]
    for c, (w, h) in enumerate(SIZES):
        s.cam_vp[c] = sg.view_proj(sg.FIXED_EYE, aspect=w / h).reshape(16)
    s = dataclasses.replace(s, smooth=look == "smooth")
    for debug in (True, False):
        with vuda.World(s, debug=debug) as w:
            w.set_tuning(vuda.TUNE_TILE_SIZE, tile)
            w.set_tuning(vuda.TUNE_RASTER_FUSED, 1 if look == "fused" else 0)
            w.step(nsteps=60)
            compare_render(w, s)
            assert any((d == 0xFFFFFFFF).any() for d in w.images(vuda.FETCH_DEPTH))
