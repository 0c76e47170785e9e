"""Shapes that share out a rod of the same size differently return the same bits: the default of
crowded handles (one wavefront of four elements per lane) against four wavefronts of one, and the
adjoint's gradients in one element per lane (its sums paired as in two) against two."""
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


def _rods(sizes, inext):
    out = []
    for k, n in enumerate(sizes):
        rng = np.random.default_rng((n, k))
        spec, st = W.straight_rod(n, L=n / 64, radius=0.005, young=1e6, inextensible=inext, damp=0.1)
        st = st.copy()
        st.v = st.v + 0.05 * rng.normal(size=st.v.shape)
        st.w = st.w + 0.3 * rng.normal(size=st.w.shape)
        st.v[0] = 0.0
        st.w[0] = 0.0
        out.append((spec, st))
    dt = min(R.stable_dt(s) for s, _ in out)
    return [(s.replace(dt=dt), st) for s, st in out]


@pytest.mark.parametrize("n,pair", [(65, ((1, 2), (2, 1))), (128, ((1, 2), (2, 1))),
                                    (129, ((2, 2), (4, 1))), (193, ((2, 2), (4, 1))),
                                    (256, ((2, 2), (4, 1))), (257, ((4, 2), (8, 1))),
                                    (511, ((4, 2), (8, 1)))])
@pytest.mark.parametrize("inext", [True, False])
def test_adjoint_shapes_return_the_same_gradients(n, pair, inext):
    import torch
    rods = _rods((n, max(n - 63, pair[0][0] * 32)), inext)
    steps, every = 12, 5
    rng = np.random.default_rng(n)
    ct = torch.from_numpy(rng.normal(size=(2, steps, 3)).astype(np.float32)).cuda()
    got = []
    for shape in pair:
        b = R.RodBatch([s for s, _ in rods])
        b.set_tuning(*shape, 10)
        b.set_state_rods([st for _, st in rods])
        tips = torch.empty((2, steps, 3), device="cuda")
        b.adjoint_forward(steps, every, tips)
        out = {q: torch.empty(m, device="cuda")
               for q, m in (("bend", 2), ("twist", 2), ("x", 3 * b.n_points), ("v", 3 * b.n_points),
                            ("q", 4 * b.n_frames), ("w", 3 * b.n_frames))}
        b.adjoint_backward(ct, out)
        b.sync()
        got.append({q: a.cpu().numpy() for q, a in out.items()})
        got[-1]["tips"] = tips.cpu().numpy()
        b.close()
    for q in got[0]:
        assert np.isfinite(got[0][q]).all() and np.abs(got[0][q]).max() > 0, q
        assert np.array_equal(got[0][q], got[1][q]), q


def test_crowded_default_is_bitwise_four_wavefronts():
    rods = _rods([129 + k % 128 for k in range(1100)], True)   # more wavefronts than SIMDs in 4 x 1
    ends, shapes = [], []
    for tuned in (False, True):
        b = R.RodBatch([s for s, _ in rods])
        if tuned:
            b.set_tuning(4, 1, 10)
        b.set_state_rods([st for _, st in rods])
        b.step(20, 10)
        b.sync()
        shapes.append({t[:2] for t in b.buckets()})
        ends.append(b.get_state_rods())
        b.close()
    assert shapes == [{(1, 4)}, {(4, 1)}]
    for a, c in zip(*ends):
        for u, v in zip(a, c):
            assert np.array_equal(np.asarray(u), np.asarray(v))
