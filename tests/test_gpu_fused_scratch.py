"""Fused frames whose records pass through the raster scratch, frame after
frame: each one rewrites the records that earlier frames left there, so a tile
that read a record before this frame's was in place would show an earlier
frame's triangle.  Bit for bit against the two-kernel path, through the C ABI.
(The build refuses a fused kernel that reads its records with scalar loads.)
"""
import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


# large triangles (the ground, cubes near the camera) and moving bodies; every
# record, or those of the larger images, in the scratch; one workgroup per
# image, or few that go over all of them
@pytest.mark.parametrize("records", [1, 150])
@pytest.mark.parametrize("persistent", [0, 7])
@pytest.mark.parametrize("tile,threads", [(16, 256), (16, 1024), (8, 512), (32, 256)])
def test_records_of_each_frame(records, persistent, tile, threads):
    s = sg.config_scene(4, n_envs=48)
    with vuda.World(s) as a, vuda.World(s) as b:
        for w in (a, b):
            w.set_tuning(vuda.TUNE_TILE_SIZE, tile)
        a.set_tuning(vuda.TUNE_RASTER_FUSED, 1)
        a.set_tuning(vuda.TUNE_FUSED_LDS_RECORDS, records)
        a.set_tuning(vuda.TUNE_RASTER_THREADS, threads)
        a.set_tuning(vuda.TUNE_RASTER_PERSISTENT, persistent)
        for frame in range(12):
            for w in (a, b):
                w.step(nsteps=1 + frame % 3)
                w.render()
                w.wait()
            for what in (vuda.FETCH_RGB, vuda.FETCH_DEPTH):
                assert np.array_equal(a.fetch(what), b.fetch(what)), f"frame {frame}"
