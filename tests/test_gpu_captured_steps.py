"""Steps captured into a graph and replayed between eager steps: rods that step as chunks also then
(longer than 2048 elements; every replay waits for its neighbours anew), and rods of an untuned
handle, whose eager steps are spread over chunks and whose captured ones are not."""
import numpy as np
import pytest

from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_iter,steps", [(4096, 0, 10), (4096, 0, 40), (9000, 10, 12), (2048, 10, 12),
                                            (700, 0, 8)])
def test_replays_are_bitwise_eager_steps(n, n_iter, steps):
    import torch
    rng = np.random.default_rng(n)
    spec, _ = W.straight_rod(n, L=n / 64.0, radius=0.01, young=1e6, inextensible=n_iter > 0, dt=1.0,
                             damp=0.1, n_iter=n_iter, clamp=True)
    x, q = W.curved_rod(n, 1.0 / 64.0, rng, sigma=0.03)
    spec = spec.replace(clamp_x0=tuple(x[0]), clamp_q0=tuple(q[0]))
    spec = spec.replace(dt=0.5 * R.stable_dt(spec))
    st = W.RodState(x, 0.1 * rng.normal(size=(n + 1, 3)), q, 0.5 * rng.normal(size=(n, 3)))
    torch.cuda.init()
    s = torch.cuda.Stream()
    other = R.RodBatch([spec], torch.cuda.Stream().cuda_stream)
    other.set_state_rods([st])
    ref = R.RodBatch([spec], s.cuda_stream)
    b = R.RodBatch([spec], s.cuda_stream)
    for h in (ref, b):
        h.set_state_rods([st])
        h.step(3, 3)
        h.sync()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        b.step(steps, steps)
    for _ in range(4):
        with torch.cuda.stream(s):
            g.replay()
        ref.step(steps, steps)
        assert all(np.array_equal(u, v) for u, v in zip(ref.get_state(), b.get_state()))
        other.step(7, 7)      # eager runs of this and another handle in between
        for h in (ref, b):
            h.step(2, 2)
        other.sync()
    for h in (other, ref, b):
        h.close()
