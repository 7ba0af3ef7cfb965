"""Contact capacity of an env of at most 64 bodies beside a larger one: a launch
has the capacities of its largest env for every env in it, 256 pairs in contact
and 512 candidate pairs where one of more than 64 bodies is among them.  Contact
sets and state against the oracle, bit for bit.
"""
import numpy as np
import pytest

import oracle
from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda
from tests.gpu_util import compare_step, oracle_step_from, state_equal

pytestmark = pytest.mark.gpu


def lattice(kinds, spacing):
    """64 bodies of 20 cm on a cubic lattice in free fall."""
    s = sg.make_scene(1980, [64], 32, mixed=False)
    s.btype[:] = {"spheres": 0, "cubes": 1, "both": np.arange(64) % 2}[kinds]
    s.size[:] = 0.1
    s.rbound[:] = np.where(s.btype == 0, 0.1, 0.1 * np.sqrt(3.0)).astype(np.float32)
    grid = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(64, 3)
    s.pos[:] = (grid * spacing + [0.0, 0.0, 1.0]).astype(np.float32)
    s.vel[:] = 0.0
    s.omega[:] = 0.0
    s.quat[:] = [1.0, 0.0, 0.0, 0.0]
    return s


# more pairs in contact, or more candidates, than a launch of envs of at most 64
# bodies has room for (128 and 256): 144 pairs in contact; 129; 360 candidates
@pytest.mark.parametrize("kinds,spacing", [("spheres", 0.195), ("both", 0.195), ("cubes", 0.205)])
@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("broadphase", [0, 1])
def test_dense_env_beside_a_larger_one(kinds, spacing, first, broadphase):
    oracle.lib()
    dense, other = lattice(kinds, spacing), sg.make_scene(1981, [65, 3], 32, mixed=True)
    s = sg.Scene.concat([dense, other] if first else [other, dense])
    with vuda.World(s, debug=True) as w:
        w.set_tuning(vuda.TUNE_BROADPHASE, broadphase)
        r = compare_step(w, s)
        assert r["bitexact"], r


# calls of several steps, which end in the buffer they began in or in the other
# one; two dense envs, or one, in a workgroup; few workgroups that go over all
@pytest.mark.parametrize("steps", [2, 3])
@pytest.mark.parametrize("persistent", [0, 1])
def test_several_steps_of_dense_envs(steps, persistent):
    oracle.lib()
    other = sg.make_scene(1982, [65, 3, 64], 32, mixed=True)
    s = sg.Scene.concat([lattice("spheres", 0.195), other, lattice("both", 0.195), lattice("cubes", 0.205)])
    ref = s.state()
    for _ in range(steps):
        ref, _ = oracle_step_from(s, ref, range(s.n_envs))
    with vuda.World(s) as w:
        w.set_tuning(vuda.TUNE_PHYS_PERSISTENT, persistent)
        w.step(nsteps=steps)
        w.wait()
        assert state_equal(w.state(), ref)
