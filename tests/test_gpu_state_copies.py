"""State copies to and from caller arrays in one launch: odd sizes, arrays that start at any 4-byte
address (whole quads only where both sides are aligned), some arrays skipped, device and host
arrays, a handle on another stream than torch's, and the start time passed with the state."""
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


def _arrays(ns, seed):
    rng = np.random.default_rng(seed)
    p, f = sum(ns) + len(ns), sum(ns)
    return [rng.normal(size=k).astype(np.float32) for k in (3 * p, 3 * p, 4 * f, 3 * f)]


def _handle(ns, stream=None):
    return R.RodBatch([W.straight_rod(n, dt=1e-6)[0] for n in ns], stream)


def _at(a, shift):
    """The array on the device, starting shift floats into an allocation."""
    import torch
    t = torch.zeros(a.size + 8, dtype=torch.float32, device="cuda")
    v = t[shift:shift + a.size]
    v.copy_(torch.from_numpy(a))
    return v


@pytest.mark.parametrize("ns", [[1], [2, 1], [63, 5], [4096, 33], [70, 71, 72, 1000]])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_round_trip(ns, shift):
    import torch
    want = _arrays(ns, 1 + shift)
    b = _handle(ns)
    b.set_state(*[_at(a, shift) for a in want])
    got = [_at(np.zeros_like(a), (shift + 1) % 4) for a in want]
    b.get_state(got)
    host = b.get_state()
    for a, d, h in zip(want, got, host):
        assert np.array_equal(a, d.cpu().numpy()) and np.array_equal(a, h)
    # one array alone, and neighbours of the written ranges untouched
    only = torch.full((want[0].size + 2,), 7.0, device="cuda")
    b.get_positions(only[1:-1])
    assert np.array_equal(only[1:-1].cpu().numpy(), want[0])
    assert only[0].item() == 7.0 and only[-1].item() == 7.0
    b.close()


def test_new_state_replaces_low_parts_and_time():
    """A rollout from a state set again is the rollout from that state: low parts, step count and
    start time start over."""
    wl = W.config1(n=64)
    b = R.RodBatch([s for s, _ in wl.rods])
    outs = []
    for t0 in (0.0, 1e-3, 0.0):
        b.set_state_rods([st for _, st in wl.rods], t0)
        b.step(40, 7)
        outs.append(b.get_state())
        assert b.time() == (t0 + 40 * wl.rods[0][0].dt, 40)
    b.close()
    assert all(np.array_equal(u, v) for u, v in zip(outs[0], outs[2]))
    assert not np.array_equal(outs[0][0], outs[1][0])   # driven clamps: the start time matters


def test_handle_on_another_stream():
    """Arrays freed right after set_state on a handle whose stream is not the current one."""
    import torch
    ns = [500, 77]
    s = torch.cuda.Stream()
    b = _handle(ns, s.cuda_stream)
    for seed in range(5):
        want = _arrays(ns, seed)
        torch.cuda.synchronize()
        dev = [torch.from_numpy(a).cuda() for a in want]
        torch.cuda.synchronize()
        b.set_state(*dev)
        del dev
        for a in want:   # reuses the freed memory on the current stream
            torch.full((a.size,), 9.0, device="cuda")
        got = b.get_state()
        assert all(np.array_equal(u, v) for u, v in zip(want, got))
    b.close()
