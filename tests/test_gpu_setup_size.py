"""Setup workgroups of 512 threads, which a launch of few images takes until a
size is set, give the frames of every size that can be asked for.  Bit for
bit, through the C ABI; and the reported size is the documented default.
"""
import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


# the last count of images that takes 512 threads and the first that does not,
# alone and co-scheduled
@pytest.mark.parametrize("envs,split", [(1, 0.0), (512, 0.0), (513, 0.0), (256, 2.0), (257, 2.0), (64, 0.5)])
def test_default_setup_size(envs, split):
    counts = ([1, 40, 7, 128] + [2] * 509)[:envs]
    s = sg.make_scene(1600 + envs, counts, 64, mixed=True)
    with vuda.World(s) as w:
        w.cosched(split)
        assert w.get_tuning(vuda.TUNE_RASTER_THREADS) == 256
        w.step(nsteps=3)
        w.render()
        w.wait()
        rgb = [a.copy() for a in w.images(vuda.FETCH_RGB)]
        dep = [a.copy() for a in w.images(vuda.FETCH_DEPTH)]
        for threads in (64, 256, 512):
            w.set_tuning(vuda.TUNE_RASTER_THREADS, threads)
            assert w.get_tuning(vuda.TUNE_RASTER_THREADS) == threads
            w.load_state(w.state())
            w.render()
            w.wait()
            for c, (a, b) in enumerate(zip(w.images(vuda.FETCH_RGB), w.images(vuda.FETCH_DEPTH))):
                assert np.array_equal(a, rgb[c]) and np.array_equal(b, dep[c]), f"image {c}, {threads} threads"
