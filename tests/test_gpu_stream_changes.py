"""Streams come and go with vuda_cosched; events of the world outlive them.  Many
changes of the split with launches of every kind in between (events recorded on
a stream, bound to launches, timing events not yet read, work lists rebuilt while
launches read them, captured graphs) keep every call succeeding and leave the
results of one stream.
"""
import numpy as np
import pytest

from paper_2605_01352_amd import scenegen as sg
from paper_2605_01352_amd import vuda

pytestmark = pytest.mark.gpu


def test_splits_change_with_events_in_use():
    s = sg.make_scene(2400, [6, 3, 12, 1] * 8, 32, mixed=True)
    splits = [2.0, 0.5, 0.0, 2.0, 0.25, 2.0, 0.75, 0.0]
    steps = 0
    with vuda.World(s) as w, vuda.World(s) as ref:
        for k in range(24):
            w.cosched(splits[k % len(splits)])
            # events recorded on the streams (timing, graphs) ...
            w.set_tuning(vuda.TUNE_TIMING, 1)
            w.set_tuning(vuda.TUNE_GRAPHS, k % 3 == 0)
            for _ in range(5):
                w.run(vuda.SCHED_INTERSTEP, 2)
            if k % 2:  # else they are read after the streams are gone
                assert w.kernel_times(vuda.KERNEL_PHYSICS)["launches"] > 0
            w.set_tuning(vuda.TUNE_TIMING, 0)
            w.set_tuning(vuda.TUNE_GRAPHS, 0)
            # ... and bound to launches, past the pool's 512
            w.run(vuda.SCHED_PIPELINED if k % 2 else vuda.SCHED_INTERTRAJ, 300)
            w.set_tuning(vuda.TUNE_TILE_WAVES, 1 + k % 2)  # the lists are rebuilt behind their fences
            w.run(vuda.SCHED_INTERSTEP, 2)
            steps += 312
            junk = [np.full(n, 0xFF, np.uint8) for n in range(64, 4096, 64)]  # memory that was freed is used again
            del junk
        w.wait()
        t = w.kernel_times(vuda.KERNEL_RASTER_TILES)
        assert t["launches"] > 0 and 0 < t["max_ms"] <= t["total_ms"]
        ref.step(nsteps=steps)
        a, b = w.state(), ref.state()
        assert all(np.array_equal(a[c].view(np.uint32), b[c].view(np.uint32)) for c in a)
