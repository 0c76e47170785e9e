"""Environment collision through the candidate and near lists against the walk of the tree.

A rod pressed into a tube is stepped twice from one state: in one run, where most steps test the
triangles near each point that are kept in LDS (or the candidate list, where more than eight are
near, or the tree, where more than 32 are candidates), and with the mesh set anew before every
step, which drops the lists, so that every step's hits come from the walk.  Both find the same
triangles and sum them in tree order, so the states are the same bits: no tolerance."""
import sys

import numpy as np
import pytest

from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.init()
    yield


def _split(tris):
    a, b, c = tris[:, 0], tris[:, 1], tris[:, 2]
    ab, bc, ca = (a + b) / 2, (b + c) / 2, (c + a) / 2
    return np.concatenate([np.stack(t, 1) for t in ((a, ab, ca), (ab, b, bc), (ca, bc, c),
                                                    (ab, bc, ca))])


# elements, triangles around the tube, splits of each into four, how far the rod lies below the
# axis (10 mm tube, 2 mm spheres: touching from 8 mm), kept as: near / candidate list / tree
CASES = [(1, 12, 0, 8.1e-3), (64, 12, 0, 8.1e-3),   # 1 x 1, one slot and a full wavefront
         (100, 24, 0, 9.0e-3),                      # 2 x 1, three to eight near
         (300, 24, 0, 9.8e-3),                      # 4 x 2, more than eight near for many points
         (700, 24, 1, 8.1e-3),                      # 4 x 4, more than 32 candidates
         (2048, 12, 0, 8.1e-3)]                     # 8 x 4, the largest rod of one workgroup


@pytest.mark.parametrize("n,around,splits,sink", CASES)
@pytest.mark.parametrize("inext", [True, False])
def test_lists_find_what_the_walk_finds(n, around, splits, sink, inext):
    centre = W.tube_centreline()
    tris = W.tube_mesh(centre, 1e-2, around)
    for _ in range(splits):
        tris = _split(tris)
    cum = np.r_[0.0, np.cumsum(np.linalg.norm(np.diff(centre, axis=0), axis=1))]
    s = np.linspace(0.3, 0.9, n + 1) * cum[-1]
    x = np.stack([np.interp(s, cum, centre[:, c]) for c in range(3)], 1)
    x[:, 2] -= sink
    rng = np.random.default_rng(n)
    v = rng.normal(size=(n + 1, 3)) * 0.05
    v[0] = 0.0
    w = rng.normal(size=(n, 3)) * 0.3
    w[0] = 0.0
    q = W.frames_from_polyline(x)
    spec = W.RodSpec(n=n, inextensible=inext, n_iter=10 if inext else 0, clamp=True, dt=1.0,
                     gravity=(0.0, 0.0, -9.81), damp_lin=0.5, damp_ang=0.5, poisson=0.5,
                     density=1000.0, seg_len=np.linalg.norm(np.diff(x, axis=0), axis=1),
                     radius=np.full(n, 2e-3), young=np.full(n, 1e7), clamp_x0=tuple(x[0]),
                     clamp_q0=tuple(q[0]))
    spec = spec.replace(dt=R.stable_dt(spec))
    st = W.RodState(x=x, v=v, q=q, w=w)
    steps = 24

    def run(calls, per_call, remesh):
        b = R.RodBatch([spec])
        b.set_environment(tris, 0.3)
        b.set_state_rods([st])
        for _ in range(calls):
            if remesh:
                b.set_environment(tris, 0.3)
            b.step(per_call, per_call)
        out = b.get_state_rods()[0]
        b.close()
        return out

    walk = run(steps, 1, True)
    free = R.RodBatch([spec])
    free.set_state_rods([st])
    free.step(steps, steps)
    plain = free.get_state_rods()[0]
    free.close()
    assert any((a != b).any() for a, b in zip(walk, plain)), "the rod never touched the mesh"
    for calls, per_call in ((1, steps), (4, steps // 4), (steps, 1)):
        print("[gpu-test] %d elements, %d triangles: %d x %d steps" % (n, len(tris), calls, per_call),
              flush=True)
        sys.stdout.flush()
        for name, a, b in zip("xvqw", run(calls, per_call, False), walk):
            assert np.array_equal(np.asarray(a), np.asarray(b)), name
