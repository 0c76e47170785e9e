"""Bound rods where the bindings at a wavefront's edge slots are applied by its neighbour too: pairs
whose bound ranges end at, before and after the wavefront boundaries of both rods, uneven lengths,
one- and two-way, against the oracle's pair step."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.init()
    yield


def _pair(na, nb, shift):
    """Two coaxial soft rods, point k + shift of the first at point k of the second."""
    l = 1.0 / 64
    rng = np.random.default_rng((na, nb, shift))
    rods = []
    for n, back in ((na, shift), (nb, 0)):
        spec, st = W.straight_rod(n, L=n * l, radius=0.005, young=1e6, inextensible=True, dt=1.0,
                                  damp=0.2)
        x = st.x + np.array([-back * l, 0.0, 0.0])
        spec = spec.replace(clamp_x0=tuple(x[0]))
        f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
        rods.append((spec, W.RodState(f32(x), f32(0.05 * rng.normal(size=x.shape)), st.q,
                                      f32(0.3 * rng.normal(size=(n, 3))))))
    dt = 0.5 * min(R.stable_dt(s) for s, _ in rods)
    return [(s.replace(dt=dt), st) for s, st in rods]


@pytest.mark.parametrize("one_way", [True, False])
@pytest.mark.parametrize("na,nb,shift,lo,hi", [
    (128, 128, 0, 1, 128),        # one wavefront each
    (129, 200, 1, 1, 127),        # two: the binding ends at the boundary
    (256, 150, 3, 126, 131),      # only around the boundary
    (300, 260, 7, 1, 252),        # four, uneven
    (512, 385, 128, 1, 384),      # a whole shape, ending one slot past a boundary
    (700, 600, 60, 500, 600),     # eight slots per lane
])
def test_bindings_at_wavefront_edges(na, nb, shift, lo, hi, one_way):
    rods = _pair(na, nb, shift)
    k = np.arange(lo, hi + 1)
    pairs = np.stack([0 * k, k + shift, 0 * k + 1, k], 1)
    pairs = pairs[pairs[:, 1] <= na].astype(np.int32)
    out = []
    for split in (1, 25):
        b = R.RodBatch([s for s, _ in rods])
        b.set_bindings(pairs, one_way)
        b.set_state_rods([st for _, st in rods])
        b.step(25, split)
        b.sync()
        out.append(b.get_state_rods())
        b.close()
    # a launch per step and one for all: the same states, so nothing is carried between steps
    assert all(np.array_equal(u, v) for a, c in zip(*out) for u, v in zip(a, c))
    ref = O.rollout_pair(rods[0][0], rods[1][0], rods[0][1], rods[1][1], pairs[:, 1], pairs[:, 3],
                         one_way, 25)
    for (spec, _), got, end in zip(rods, out[1], ref):
        err = np.abs(got[0] - end.x).max()
        tol = 1e-4 * float(np.sum(spec.seg_len))   # the method's position target
        print("%d/%d %s: max|dx| %.2e (tol %.1e)" % (na, nb, "one" if one_way else "two", err, tol),
              flush=True)
        assert err <= tol
    if not one_way:   # bound points end every step together
        pa, pb = out[1][0][0][pairs[:, 1]], out[1][1][0][pairs[:, 3]]
        assert np.abs(pa - pb).max() <= 1e-6
