"""More chunks in flight than the device has compute units, from two host threads: handles of long
rods, whose runs then wait for each other, and untuned handles of shorter ones, which step in one
workgroup per rod instead; launches with many halo exchanges and with none.  The states are
bitwise those of each handle alone."""
import threading

import numpy as np
import pytest

from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


def _rod(n):
    rng = np.random.default_rng(n)
    spec, _ = W.straight_rod(n, L=n / 64.0, radius=0.01, young=1e6, inextensible=True, dt=1.0,
                             damp=0.1, n_iter=10, clamp=True)
    x, q = W.curved_rod(n, 1.0 / 64.0, rng, sigma=0.03)
    spec = spec.replace(clamp_x0=tuple(x[0]), clamp_q0=tuple(q[0]))
    spec = spec.replace(dt=0.5 * R.stable_dt(spec))
    return spec, W.RodState(x, 0.1 * rng.normal(size=(n + 1, 3)), q, 0.5 * rng.normal(size=(n, 3)))


@pytest.mark.parametrize("sizes", [[2048 - 8 * i for i in range(28)],
                                   [17000 + 100 * i for i in range(4)],
                                   [17000, 2048, 2000, 17100, 1500, 17200] + [1900 - 8 * i for i in range(10)]])
@pytest.mark.parametrize("splits", [[20, 20, 20], [2] * 15])
def test_handles_in_flight_together(sizes, splits):
    import torch
    torch.cuda.init()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rods = [_rod(n) for n in sizes]
    alone = []
    for spec, st in rods:
        b = R.RodBatch([spec])
        b.set_state_rods([st])
        for k in splits:
            b.step(k, k)
        b.sync()
        alone.append(b.get_state())
        b.close()
    streams = [torch.cuda.Stream() for _ in rods]
    hs = [R.RodBatch([spec], s.cuda_stream) for (spec, _), s in zip(rods, streams)]
    for h, (_, st) in zip(hs, rods):
        h.set_state_rods([st])
    assert sum(h.chunks[0] for h in hs) > cus
    torch.cuda.synchronize()

    def drive(part):
        for k in splits:
            for h in part:
                h.step(k, k)

    threads = [threading.Thread(target=drive, args=(p,)) for p in (hs[::2], hs[1::2])]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for h, want in zip(hs, alone):
        h.sync()
        assert all(np.array_equal(u, v) for u, v in zip(want, h.get_state()))
    for h in hs:
        h.close()
