"""GPU parity of layer 1's stages of 32 and 64 observation values and of the
head's one and two envs per workgroup, through the C ABI, at ragged batches,
hidden sizes and chunk counts.

Gate: the oracle's float32 error bound on the actions (as in
test_gpu_policy.py), on frames checked to be identical.
"""
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda
from tests.test_gpu_policy import check_actions

pytestmark = pytest.mark.gpu


# frame, envs, hidden: frames of 32 and of an odd multiple of 32 pixels (stages
# of 32), one chunk of 4 stages (8x4); stages of 64, one chunk (8x8) and 128
# (64x64), with chunks that start in the depth part, hold its start and lie in
# the RGB part; whole RGB stages in chunks of 27 steps of 32 (24x72)
@pytest.mark.parametrize("width,height,envs,hidden", [
    (8, 4, 3, 5), (12, 8, 65, 300), (36, 24, 130, 257), (8, 8, 64, 256), (64, 64, 1, 1), (64, 64, 67, 513),
    (24, 72, 3, 64)])
def test_layer1_stages(width, height, envs, hidden):
    s = sg.make_scene(1300 + envs, [2] * envs, 64, mixed=True)
    s.cam_w[:] = width
    s.cam_h[:] = height
    P = sg.policy_weights(31, width, height, hidden, 2)
    with vuda.World(s) as w:
        w.step(nsteps=5)
        w.set_policy(P)
        check_actions(w, s, P, range(s.n_envs), f"policy {envs} envs {width}x{height} H{hidden}")


# two envs per workgroup (at least 2^18 hidden units over the batch): an odd
# batch, a hidden size that is no multiple of 4 or of 64, more and fewer
# actions than lanes; and the last batch that takes one
@pytest.mark.parametrize("envs,hidden,bodies", [(257, 1024, 2), (513, 515, 40), (512, 513, 1), (511, 512, 3)])
def test_head_envs_per_workgroup(envs, hidden, bodies):
    s = sg.make_scene(1700 + envs, [bodies] * envs, 8, mixed=True)
    P = sg.policy_weights(33, 8, 8, hidden, bodies)
    with vuda.World(s) as w:
        w.step(nsteps=5)
        w.set_policy(P)
        check_actions(w, s, P, [0, 1, 63, 64, envs - 2, envs - 1], f"policy {envs} envs H{hidden}")
