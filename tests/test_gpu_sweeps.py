"""Constraint iterations and exchanges of the step kernels where their forms differ: every count
of iterations modulo the unrolled four, clamped and free bases, rods that end just before, at
and just after a lane's, a wavefront's and a shape's last slot, in every shape that holds them
(one wavefront takes its neighbour's impulse, several evaluate it; one slot per lane evaluates
only the segment it takes part in)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 2), (1, 4), (1, 8), (2, 1), (2, 2), (2, 4), (4, 1), (4, 2), (4, 4), (4, 8),
          (8, 1), (8, 2), (8, 4), (16, 1)]


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.init()
    yield


def _rod(n, n_iter, clamp, inext=True):
    """A curved moving rod with uneven segments and an external load."""
    rng = np.random.default_rng((n, n_iter))
    spec, st = W.straight_rod(n, L=n / 64.0, radius=0.01, young=1e6, inextensible=inext, dt=1.0,
                              damp=0.1, n_iter=n_iter, clamp=clamp)
    x, q = W.curved_rod(n, 1.0 / 64.0, rng, sigma=0.03)
    seg = np.linalg.norm(np.diff(x, axis=0), axis=1) * (1 + 1e-4 * rng.normal(size=n))
    spec = spec.replace(seg_len=seg, clamp_x0=tuple(x[0]), clamp_q0=tuple(q[0]),
                        f_ext=1e-3 * rng.normal(size=(n + 1, 3)))
    spec = spec.replace(dt=0.5 * R.stable_dt(spec))
    f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
    return spec, W.RodState(f32(x), f32(0.1 * rng.normal(size=(n + 1, 3))), f32(q),
                            f32(0.5 * rng.normal(size=(n, 3))))


def _run(rod, steps, shape):
    b = R.RodBatch([rod[0]])
    b.set_tuning(*shape, 7)
    b.set_state_rods([rod[1]])
    b.step(steps, 7)
    b.sync()
    out = b.get_state()
    b.close()
    return out


@pytest.mark.parametrize("n_iter,clamp", [(0, True), (1, True), (2, False), (3, True), (4, False),
                                          (5, True), (7, False), (10, True)])
@pytest.mark.parametrize("n", [1, 2, 3, 64, 65, 127, 128, 130, 257])
def test_iterations_in_every_shape(n, n_iter, clamp):
    rod = _rod(n, n_iter, clamp)
    shapes = [s for s in SHAPES if 64 * s[0] * s[1] >= n]
    ref = _run(rod, 20, shapes[0])
    for s in shapes[1:]:
        got = _run(rod, 20, s)
        assert all(np.array_equal(a, b) for a, b in zip(ref, got)), s
    end, _ = O.Rod(rod[0]).rollout(rod[1], 20)
    err = np.abs(ref[0].reshape(-1, 3) - end.x).max()
    tol = 1e-4 * float(np.sum(rod[0].seg_len))   # the method's position target
    print("n %d iterations %d clamp %d: max|dx| %.2e (tol %.1e)" % (n, n_iter, clamp, err, tol), flush=True)
    assert err <= tol
