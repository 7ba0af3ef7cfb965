"""Runs of tiles per wave: a list of many tiles, whose waves go over several
tiles of a row each, gives the frames that short lists of the same images
give, where every wave takes one tile.  Bit for bit, through the C ABI.
"""
import dataclasses

import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


# 8-pixel tiles: 180 images of up to 256 tiles, over 40,000 in all, so that the
# first ones (the largest, then by id) are in runs of 2 or 8 tiles and the last
# 28,672 tiles in single ones; rows of 1, 2, 3, 5, 9, 13, 15 and 16 tiles
@pytest.mark.parametrize("waves", [1, 2, 4])
@pytest.mark.parametrize("smooth", [False, True])
def test_tile_runs(waves, smooth):
    s = sg.make_scene(1500, [6, 1, 11] * 60, 128, mixed=True)
    for i, (w, h) in enumerate([(8, 128), (16, 61), (20, 100), (36, 16), (72, 72), (100, 61), (113, 128), (7, 7)]):
        s.cam_w[3 + 20 * i] = w
        s.cam_h[3 + 20 * i] = h
    s = dataclasses.replace(s, smooth=smooth)
    with vuda.World(s) as w:
        w.set_tuning(vuda.TUNE_TILE_SIZE, 8)
        w.set_tuning(vuda.TUNE_TILE_WAVES, waves)
        w.step(nsteps=5)
        tiles = int((((s.cam_w.astype(int) + 7) // 8) * ((s.cam_h.astype(int) + 7) // 8)).sum())
        assert tiles > 40000
        w.render()
        w.wait()
        rgb, dep = w.images(vuda.FETCH_RGB), w.images(vuda.FETCH_DEPTH)
        rgb, dep = [a.copy() for a in rgb], [a.copy() for a in dep]
        w.load_state(w.state())
        for e in range(0, s.n_envs, 30):
            w.render(e, e + 30)
        w.wait()
        for c, (a, b) in enumerate(zip(w.images(vuda.FETCH_RGB), w.images(vuda.FETCH_DEPTH))):
            assert np.array_equal(a, rgb[c]) and np.array_equal(b, dep[c]), f"image {c}"
        assert sum((d != 0xFFFFFFFF).any() for d in dep) > 170
        say(f"{tiles} tiles, {waves} waves per workgroup: frames equal")
