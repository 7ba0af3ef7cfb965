"""The forced grid broadphase in envs of 33 to 64 bodies when a body leaves the
grid's range (1,000 cells from the origin) between two substeps: the later
substeps look at all pairs, and keep every contact.  Contact sets and state
against the oracle, bit for bit.
"""
import numpy as np
import pytest

import oracle
from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda
from tests.gpu_util import compare_step, oracle_step_from, say, state_equal

pytestmark = pytest.mark.gpu


def straddling_pile(bodies, substeps_ahead):
    """Settled piles moved along x so that the foremost body, at 4 m/s, passes
    cell 1,000 half way through the given substep (0 the first)."""
    s = sg.make_scene(1900 + bodies, [bodies, bodies], 32, mixed=True)
    with vuda.World(s) as w:
        w.step(nsteps=300)
        w.wait()
        st = w.state()
    speed, h = 4.0, s.dt / s.substeps
    for e in range(s.n_envs):
        b = slice(int(s.body_off[e]), int(s.body_off[e + 1]))
        edge = 1000.0 * 2.0 * float(s.rbound[b].max()) * 1.000244140625
        front = b.start + int(st["pos"][b, 0].argmax())
        st["pos"][b, 0] += np.float32(edge - speed * h * (substeps_ahead + 0.5)) - st["pos"][front, 0]
        st["vel"][front] = [speed, 0.0, 0.0]
    return s, st


@pytest.mark.parametrize("bodies", [33, 48, 64])
@pytest.mark.parametrize("beside", [0, 100])
@pytest.mark.parametrize("substep", [0, 2])
def test_body_leaves_the_grid_mid_step(bodies, beside, substep):
    oracle.lib()
    s, st = straddling_pile(bodies, substep)
    if beside:  # an env of two waves in the same launch
        o = sg.make_scene(1950, [beside], 32, mixed=True)
        st = {k: np.concatenate([st[k], o.state()[k]]) for k in st}
        s = sg.Scene.concat([s, o])
    with vuda.World(s, debug=True) as w:
        w.set_tuning(vuda.TUNE_BROADPHASE, 1)
        w.load_state(st)
        r = compare_step(w, s)
        assert r["bitexact"], r
        assert any((c[:, 1] != 0xFFFF).any() for e in w.contacts()[:2] for c in e[1:])  # bodies in contact
    say(f"{bodies} bodies, past the grid in substep {substep}: contact sets equal")


@pytest.mark.parametrize("bodies", [40, 64])
def test_body_leaves_the_grid_in_a_later_step_of_a_call(bodies):
    oracle.lib()
    s, st = straddling_pile(bodies, 2 * 4 + 1)
    ref = st
    for _ in range(4):
        ref, _ = oracle_step_from(s, ref, range(s.n_envs))
    with vuda.World(s) as w:
        w.set_tuning(vuda.TUNE_BROADPHASE, 1)
        w.load_state(st)
        w.step(nsteps=4)
        w.wait()
        assert state_equal(w.state(), ref)
