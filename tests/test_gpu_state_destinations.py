"""State fetches into device destinations that a kernel of the world's GPU does
not write itself: rows off whole words, and memory of another kind.
"""
import ctypes as C

import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["device", "device, off by one byte", "device, off by two", "pinned host"])
@pytest.mark.parametrize("split", [0.0, 2.0])
def test_state_into(where, split):
    import torch
    s = sg.make_scene(2000, [7, 0, 32, 100] * 3, 32, mixed=True)
    off = {"device, off by one byte": 1, "device, off by two": 2}.get(where, 0)
    with vuda.World(s) as w:
        w.cosched(split)
        w.step(nsteps=3)
        w.wait()
        host = w.fetch(vuda.FETCH_STATE)
        if where == "pinned host":
            buf = torch.full((host.nbytes + 16,), 0x5A, dtype=torch.uint8, pin_memory=True)
        else:
            buf = torch.full((host.nbytes + 16,), 0x5A, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        vuda.check(vuda.lib().vuda_fetch(w._w, vuda.FETCH_STATE, 0, w.n_envs, C.c_void_p(buf.data_ptr() + off),
                                         C.c_size_t(host.nbytes), 1))
        got = buf.cpu().numpy()
        assert np.array_equal(got[off:off + host.nbytes], host.view(np.uint8).reshape(-1))
        assert (got[:off] == 0x5A).all() and (got[off + host.nbytes:] == 0x5A).all()


def test_transfers_of_growing_and_shrinking_ranges():
    """Loads and fetches of one world whose sizes go up and down: each is whole,
    whatever staging the ones before it left."""
    counts = [1, 100, 3, 128, 0, 128, 64] * 6
    s = sg.make_scene(2001, np.minimum(counts, 40), 32, mixed=False)
    off, rng = s.body_off, np.random.default_rng(5)
    with vuda.World(s) as w:
        ref = w.fetch(vuda.FETCH_STATE).reshape(-1, 13)
        for lo, hi in [(0, 1), (0, 2), (1, 4), (0, 7), (4, 5), (0, 20), (3, 9), (0, 42), (41, 42)]:
            b = slice(int(off[lo]), int(off[hi]))
            ref[b] = rng.normal(size=ref[b].shape).astype(np.float32)
            w.load_state(vuda.aos_to_state(ref[b].copy()), lo, hi)
            assert np.array_equal(w.fetch(vuda.FETCH_STATE, lo, hi).reshape(-1, 13), ref[b])
            assert np.array_equal(w.fetch(vuda.FETCH_STATE).reshape(-1, 13), ref)
