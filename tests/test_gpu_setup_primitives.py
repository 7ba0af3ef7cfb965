"""The default setup size around the primitive counts where it changes gives the
frames of every size that can be asked for.  Bit for bit, through the C ABI.
"""
import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


# spheres of 80 faces and cubes of 12 on a ground of 2: either side of 256, 512
# and 1,024 primitives (3, 4, 6, 7 and 12, 13 spheres), at 256 images and more
@pytest.mark.parametrize("bodies", [1, 3, 4, 6, 7, 12, 13])
@pytest.mark.parametrize("envs,split", [(256, 0.0), (257, 0.0), (256, 2.0)])
def test_default_size_by_primitives(bodies, envs, split):
    s = sg.make_scene(2300 + bodies, [bodies] * envs, 64, mixed=False)
    with vuda.World(s) as w:
        w.cosched(split)
        w.step(nsteps=3)
        w.render()
        w.wait()
        rgb, dep = w.fetch(vuda.FETCH_RGB), w.fetch(vuda.FETCH_DEPTH)
        for threads in (256, 512):
            w.set_tuning(vuda.TUNE_RASTER_THREADS, threads)
            w.load_state(w.state())
            w.render()
            w.wait()
            assert np.array_equal(rgb, w.fetch(vuda.FETCH_RGB)) and np.array_equal(dep, w.fetch(vuda.FETCH_DEPTH))
