"""Every body of an env on the ground, up to the largest env: the counts of
ground contacts fill their fields in the step's packed scan.  Contact sets and
state against the oracle, bit for bit.
"""
import numpy as np
import pytest

import oracle
from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda
from tests.gpu_util import compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bodies", [32, 64, 127, 128])
@pytest.mark.parametrize("cubes", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("pack", [1, 2])
def test_all_bodies_on_the_ground(bodies, cubes, pack):
    oracle.lib()
    s = sg.make_scene(1990, [bodies] * 3, 32, mixed=False)
    i = np.arange(s.n_bodies) % bodies
    s.btype[:] = i < cubes * bodies
    s.size[:] = 0.1
    s.rbound[:] = np.where(s.btype == 0, 0.1, 0.1 * np.sqrt(3.0)).astype(np.float32)
    s.pos[:] = np.stack([i % 12 * 0.5, i // 12 * 0.5, np.full(len(i), 0.099)], -1).astype(np.float32)
    s.quat[:] = [1.0, 0.0, 0.0, 0.0]
    s.vel[:] = 0.0
    s.omega[:] = 0.0
    with vuda.World(s, debug=True) as w:
        w.set_tuning(vuda.TUNE_PHYS_ENVS_PER_WAVE, pack)
        r = compare_step(w, s)
        assert r["bitexact"], r
        assert all(len(c) == bodies and (c[:, 1] == 0xFFFF).all() for e in w.contacts() for c in e)
