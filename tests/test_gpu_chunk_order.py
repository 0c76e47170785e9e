"""Launches of chunked rods that hold no halo exchange (at most as many steps as lie between two):
a chunk stores its slots over those its neighbours load at the start of the launch, so it has to
wait until they have.  A batch on another stream keeps the compute units busy meanwhile, so that
the chunks of a launch start apart.  The states are bitwise those of one long launch alone, whose
exchanges order the chunks."""
import numpy as np
import pytest

from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def filler():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.init()
    spec, st = W.straight_rod(1000, dt=1e-6, inextensible=True)
    s = torch.cuda.Stream()
    b = R.RodBatch([spec] * 1500, s.cuda_stream)
    b.set_state_rods([st] * 1500)
    yield b
    b.close()


def _rod(n, n_iter):
    rng = np.random.default_rng((n, n_iter))
    spec, _ = W.straight_rod(n, L=n / 64.0, radius=0.01, young=1e6, inextensible=n_iter > 0, dt=1.0,
                             damp=0.1, n_iter=n_iter, clamp=True)
    x, q = W.curved_rod(n, 1.0 / 64.0, rng, sigma=0.03)
    spec = spec.replace(clamp_x0=tuple(x[0]), clamp_q0=tuple(q[0]))
    spec = spec.replace(dt=0.5 * R.stable_dt(spec))
    return spec, W.RodState(x, 0.1 * rng.normal(size=(n + 1, 3)), q, 0.5 * rng.normal(size=(n, 3)))


# (elements, iterations, chunk elements or None: the library's own choice): windows that exchange
# every step and every few, short chunks, and the kernel of one window per chunk (20 iterations)
@pytest.mark.parametrize("n,n_iter,chunk", [(2048, 10, None), (700, 0, None), (4096, 0, None),
                                            (9000, 10, None), (900, 3, 60), (600, 20, 0)])
def test_short_launches_beside_other_work(filler, n, n_iter, chunk):
    import torch
    spec, st = _rod(n, n_iter)
    splits = [1, 1, 2, 3, 1, 5, 4, 1, 2]
    outs = []
    for parts in ([sum(splits) + 41], splits + [41]):
        s = torch.cuda.Stream()
        b = R.RodBatch([spec], s.cuda_stream)
        if chunk is not None:
            b.set_chunking(32, chunk)
        b.set_state_rods([st])
        torch.cuda.synchronize()
        for k in parts:
            if len(parts) > 1:
                filler.step(40, 40)
            b.step(k, k)
        b.sync()
        outs.append(b.get_state())
        b.close()
        filler.sync()
    assert all(np.array_equal(u, v) for u, v in zip(*outs))
