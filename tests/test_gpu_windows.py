"""Chunked rods whose wavefronts step windows of their own: rods that end around a window's,
a workgroup's and a chunk's last slot, iteration counts on both sides of where the windows'
halos fit (19), exchanges every step (velocities only) and every few (whole states), short chunks
whose slots both neighbours need, free, clamped and driven bases, external loads.  The states are
bitwise those of one workgroup per rod."""
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


def _rod(n, n_iter, base):
    rng = np.random.default_rng((n, n_iter))
    spec, st = W.straight_rod(n, L=n / 64.0, radius=0.01, young=1e6, inextensible=n_iter > 0, dt=1.0,
                              damp=0.1, n_iter=n_iter, clamp=base != "free")
    x, q = W.curved_rod(n, 1.0 / 64.0, rng, sigma=0.03)
    spec = spec.replace(clamp_x0=tuple(x[0]), clamp_q0=tuple(q[0]),
                        f_ext=1e-3 * rng.normal(size=(n + 1, 3)))
    dt = 0.5 * R.stable_dt(spec)
    if base == "driven":
        spec = spec.replace(clamp_amp=(1e-3, 0.0, 0.0), clamp_twist_amp=0.1, clamp_freq=1 / (80 * dt))
    return (spec.replace(dt=dt),
            W.RodState(x, 0.1 * rng.normal(size=(n + 1, 3)), q, 0.5 * rng.normal(size=(n, 3))))


def _run(rods, splits, chunk=None, shape=None, stream=None):
    b = R.RodBatch([s for s, _ in rods], stream)
    if chunk is not None:
        b.set_chunking(32, chunk)
    if shape is not None:
        b.set_tuning(*shape, 10)
    b.set_state_rods([st for _, st in rods])
    for k in splits:
        b.step(k, k)
    b.sync()
    out = b.get_state()
    b.close()
    return out


@pytest.mark.parametrize("n,n_iter,base,chunk", [
    (33, 10, "clamped", 0), (128, 10, "free", 0), (129, 10, "driven", 0), (209, 10, "clamped", 0),
    (367, 10, "free", 0), (368, 10, "clamped", 0), (369, 10, "driven", 0), (700, 10, "clamped", 0),
    (2048, 10, "clamped", 0), (1500, 10, "free", 120), (1111, 10, "driven", 50),
    (130, 0, "free", 0), (404, 0, "clamped", 0), (405, 0, "driven", 0), (2000, 0, "clamped", 40),
    (1999, 0, "free", 14), (900, 1, "clamped", 0), (901, 3, "driven", 0), (800, 3, "free", 60),
    (1000, 15, "clamped", 0), (1001, 19, "free", 0), (600, 20, "clamped", 0), (560, 30, "driven", 0),
])
def test_windows_are_bitwise_one_workgroup(n, n_iter, base, chunk):
    rods = [_rod(n, n_iter, base)]
    ref = _run(rods, [97], shape=(8, 4))
    for splits in ([97], [1, 16, 5, 33, 42]):
        got = _run(rods, splits, chunk)
        assert all(np.array_equal(a, b) for a, b in zip(ref, got)), splits


def test_windows_of_rods_with_different_exchanges():
    """Extensible and inextensible long rods in one handle share a launch (whole-state exchanges)."""
    rods = [_rod(1200, 0, "clamped"), _rod(1300, 10, "driven"), _rod(60, 10, "free"), _rod(700, 3, "free")]
    ref, got = _run(rods, [60], shape=(8, 4)), _run(rods, [7, 53], 0)
    assert all(np.array_equal(a, b) for a, b in zip(ref, got))


@pytest.mark.parametrize("sizes", [
    [(129, 10)], [(256, 10), (257, 10)], [(368, 5)], [(369, 10), (512, 10)], [(1023, 10)],
    [(2048, 10), (513, 12), (130, 7)], [(257, 0)], [(404, 0), (300, 2)], [(405, 0)], [(513, 0), (2047, 1)],
    [(128, 10), (700, 10)], [(600, 20)],
])
def test_untuned_handles_are_bitwise_one_workgroup(sizes):
    """Handles whose shapes are left to the library, around the sizes where it spreads their rods
    over windows, against an explicit shape."""
    rods = [_rod(n, it, base) for (n, it), base in zip(sizes, ("driven", "free", "clamped"))]
    ref = _run(rods, [50], shape=(8, 4))
    for splits in ([50], [1] * 9 + [41]):
        got = _run(rods, splits)
        assert all(np.array_equal(a, b) for a, b in zip(ref, got))


def test_untuned_handles_on_many_streams():
    """Several spread handles in flight together, more chunks than compute units in all, from two
    host threads; then one of them changes over to another kernel and back."""
    import threading
    import torch
    cases = [[_rod(2048 - 8 * i, 10, "clamped")] for i in range(14)]
    refs = [_run(r, [40], shape=(8, 4)) for r in cases]
    streams = [torch.cuda.Stream() for _ in cases]
    hs = [R.RodBatch([s for s, _ in r], st.cuda_stream) for r, st in zip(cases, streams)]
    for h, r in zip(hs, cases):
        h.set_state_rods([st for _, st in r])

    def drive(part):
        for _ in range(8):
            for h in part:
                h.step(5, 5)

    ts = [threading.Thread(target=drive, args=(p,)) for p in (hs[::2], hs[1::2])]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for h, ref in zip(hs, refs):
        h.sync()
        assert all(np.array_equal(a, b) for a, b in zip(ref, h.get_state()))
    h, r = hs[0], cases[0]
    h.set_state_rods([st for _, st in r])
    h.step(15, 15)
    far = np.array([[[0, 0, -90], [1, 0, -90], [0, 1, -90]]], float)
    h.set_environment(far, 0.1)      # a mesh out of reach: the resident kernel with its code
    h.step(10, 10)
    h.set_environment(np.zeros((0, 3, 3)), 0.0)
    h.step(15, 5)
    assert all(np.array_equal(a, b) for a, b in zip(refs[0], h.get_state()))
    for h in hs:
        h.close()
