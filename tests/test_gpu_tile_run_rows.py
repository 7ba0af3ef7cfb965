"""Runs of tiles over rows of every length: frames of a list of many tiles, in
runs, whole ones of an image before the ends of its rows, are those of short
lists of the same images, a tile a wave.  Bit for bit, through the C ABI.
"""
import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


# over 40,000 tiles of 16 pixels in rows of 6 to 33, either side of the rule's
# limits of 8 and 12, with no end, ends shorter than a workgroup and longer ones
@pytest.mark.parametrize("tile,waves", [(16, 1), (16, 2), (16, 4), (8, 2), (32, 2)])
def test_rows_of_every_length(tile, waves):
    s = sg.make_scene(2200, [8, 3, 20, 1] * 30, 64, mixed=True)
    for c in range(s.n_cams):
        s.cam_w[c] = 16 * (6 + c % 28) - (c % 5) * 3
        s.cam_h[c] = 280 + c % 60
        s.cam_vp[c] = sg.view_proj(sg.FIXED_EYE, aspect=s.cam_w[c] / s.cam_h[c]).reshape(16)
    with vuda.World(s) as w:
        w.set_tuning(vuda.TUNE_TILE_SIZE, tile)
        w.set_tuning(vuda.TUNE_TILE_WAVES, waves)
        w.step(nsteps=60)
        tiles = int((((s.cam_w.astype(int) + 15) // 16) * ((s.cam_h.astype(int) + 15) // 16)).sum())
        assert tiles > 40000
        w.render()
        w.wait()
        long = w.fetch(vuda.FETCH_RGB), w.fetch(vuda.FETCH_DEPTH)
        w.load_state(w.state())
        for e in range(0, s.n_envs, 20):
            w.render(e, e + 20)
        w.wait()
        assert np.array_equal(long[0], w.fetch(vuda.FETCH_RGB))
        assert np.array_equal(long[1], w.fetch(vuda.FETCH_DEPTH))
