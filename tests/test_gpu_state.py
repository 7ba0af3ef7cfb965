"""State rows in and out of a world: what is loaded comes back bit for bit,
whichever way the rows are handed over, over ranges, parities and sizes at the
edges of the kernels' blocks and of the pinned staging; flags stay raised
until the state is loaded again."""
import ctypes as C

import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


def world_of(counts):
    counts = np.asarray(counts)
    scene = sg.make_scene(7, np.minimum(counts, 8), 64, mixed=True, cams_per_env=0)
    if (counts > 8).any():  # more bodies than placement draws quickly: far apart on a line
        B = int(counts.sum())
        one = np.ones(B, np.float32)
        scene = sg.Scene(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), np.zeros(B, np.uint8), 0.1 * one,
                         0.1 * one, one, one, np.zeros(B, np.uint8), np.zeros((B, 3), np.float32),
                         np.zeros((B, 3), np.float32), np.tile(np.array([1, 0, 0, 0], np.float32), (B, 1)),
                         np.zeros((B, 3), np.float32), np.zeros(len(counts) + 1, np.int32),
                         np.zeros((0, 16), np.float32), np.zeros(0, np.int32), np.zeros(0, np.int32))
    return vuda.World(scene), scene


def random_state(n, seed):
    r = np.random.default_rng(seed)
    st = {k: r.normal(size=(n, w)).astype(np.float32) for k, w in (("pos", 3), ("vel", 3), ("quat", 4), ("omega", 3))}
    st["quat"] /= np.linalg.norm(st["quat"], axis=1, keepdims=True)
    return st


def same(a, b):
    return all(np.array_equal(a[k].view(np.uint32), b[k].view(np.uint32)) for k in b)


# one body; either side of a 256-body block; uneven envs with an empty one;
# more than the pinned staging holds (322,638 rows)
@pytest.mark.parametrize("counts", [[1], [51] * 5, [64] * 4, [128, 128, 1], [3, 0, 7, 128, 5], [128] * 2600])
@pytest.mark.parametrize("split", [0.0, 2.0])
def test_rows_round_trip(counts, split):
    import torch
    w, scene = world_of(counts)
    off, n = scene.body_off, scene.n_bodies
    with w:
        w.cosched(split)
        st = random_state(n, 1)
        w.load_state(st)                                    # four arrays
        assert same(w.state(), st)
        rows = np.ascontiguousarray(vuda.state_to_aos(random_state(n, 2)))
        vuda.check(vuda.lib().vuda_load_state(w._w, 0, w.n_envs, rows.ctypes.data_as(C.c_void_p),
                                              C.c_size_t(rows.nbytes)))  # rows
        assert np.array_equal(w.fetch(vuda.FETCH_STATE).view(np.uint32), rows.reshape(-1).view(np.uint32))
        dev = torch.zeros(13 * n, dtype=torch.float32, device="cuda")
        w.fetch(vuda.FETCH_STATE, out=dev)
        assert np.array_equal(dev.cpu().numpy().view(np.uint32), rows.reshape(-1).view(np.uint32))
        if len(counts) > 1:
            # envs of both parities in one range
            w.step(1, w.n_envs)
            w.load_state(st)
            assert same(w.state(), st)
            lo, hi = 1, len(counts)
            part = random_state(int(off[hi] - off[lo]), 3)
            w.load_state(part, lo, hi)
            assert same(w.state(lo, hi), part)
            assert same(w.state(0, lo), {k: v[:off[lo]] for k, v in st.items()})


def test_short_state_is_refused():
    w, scene = world_of([8, 8])
    with w:
        before = w.state()
        with pytest.raises(vuda.VudaError) as e:
            w.load_state(random_state(15, 4))
        assert e.value.code == vuda.EINVAL
        assert same(w.state(), before)


@pytest.mark.parametrize("split", [0.0, 2.0])
def test_flag_stays_until_the_state_is_loaded(split):
    w, scene = world_of([8] * 70)
    with w:
        w.cosched(split)
        w.step()
        w.wait()
        good = w.state()
        bad = {k: v.copy() for k, v in good.items()}
        bad["vel"][8 * 69 + 3, 1] = np.nan
        w.load_state(bad)
        w.step()
        for _ in range(2):
            with pytest.raises(vuda.VudaError) as e:
                w.wait()
            assert e.value.code == vuda.ENUMERIC and "69" in str(e.value)
        assert w.fetch(vuda.FETCH_FLAGS)[69] == 1
        w.load_state({k: v[:8] for k, v in good.items()}, 0, 1)  # another env: the flag stays
        with pytest.raises(vuda.VudaError):
            w.wait()
        w.load_state(good)
        w.wait()
        w.step()
        w.wait()
        assert not w.fetch(vuda.FETCH_FLAGS).any()
