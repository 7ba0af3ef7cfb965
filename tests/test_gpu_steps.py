"""Several steps in one call: the state, contact sets and frames after
step(nsteps=k) are those of k single steps, whichever launches carry them."""
import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


def scene_of(sizes):
    return sg.make_scene(11, np.asarray(sizes), 32, mixed=True)


# one and two launches (64 steps a launch), even and odd ends, envs of up to
# 32, 64 and 128 bodies
@pytest.mark.parametrize("sizes", [[7, 32, 1], [40, 64, 9], [128, 65, 5, 64]])
@pytest.mark.parametrize("steps", [2, 3, 64, 65, 130])
@pytest.mark.parametrize("split", [0.0, 2.0])
def test_steps_in_one_call(sizes, steps, split):
    scene = scene_of(sizes)
    with vuda.World(scene, debug=True) as a, vuda.World(scene, debug=True) as b:
        a.cosched(split)
        b.cosched(split)
        for w in (a, b):
            w.step(nsteps=30)  # off the spawn
            w.render()         # a render of the buffer an even count of steps ends in
        a.step(nsteps=steps)
        a.render()
        for _ in range(steps):
            b.step()
        b.render()
        a.wait()
        b.wait()
        sa, sb = a.state(), b.state()
        assert all(np.array_equal(sa[k].view(np.uint32), sb[k].view(np.uint32)) for k in sa)
        for x, y in zip(a.contacts(), b.contacts()):
            assert all(np.array_equal(p, q) for p, q in zip(x, y))
        for what in (vuda.FETCH_RGB, vuda.FETCH_DEPTH):
            assert np.array_equal(a.fetch(what), b.fetch(what))


@pytest.mark.parametrize("key,value", [(vuda.TUNE_GRAPHS, 1), (vuda.TUNE_PHYS_PERSISTENT, 2),
                                       (vuda.TUNE_PHYS_ENVS_PER_WAVE, 2), (vuda.TUNE_TIMING, 1)])
def test_steps_in_one_call_under_launch_modes(key, value):
    scene = scene_of([7, 32, 1, 20, 5])
    with vuda.World(scene) as a, vuda.World(scene) as b:
        a.set_tuning(key, value)
        for k in (3, 1, 3, 2, 2, 3):
            a.step(nsteps=k)
            for _ in range(k):
                b.step()
            sa, sb = a.state(), b.state()
            assert all(np.array_equal(sa[c].view(np.uint32), sb[c].view(np.uint32)) for c in sa)


# workgroups of two waves: one env of more than 64 bodies or two smaller ones
# (an odd one left over, none at all, an empty env among them)
@pytest.mark.parametrize("sizes", [[128, 65, 64, 1, 33], [66], [65, 64], [3, 100, 0, 17, 70, 64, 32]])
@pytest.mark.parametrize("options", [{}, dict(mu=0.5, edge_contacts=True)])
@pytest.mark.parametrize("persistent", [0, 1, 3])
def test_envs_of_one_and_two_waves_together(sizes, options, persistent):
    import dataclasses

    from tests.gpu_util import compare_step
    scene = dataclasses.replace(sg.with_boxes(scene_of(sizes)), **options)
    with vuda.World(scene, debug=True) as w:
        w.set_tuning(vuda.TUNE_PHYS_PERSISTENT, persistent)
        w.step(nsteps=60)
        for _ in range(2):
            r = compare_step(w, scene)
            assert r["bitexact"], r
