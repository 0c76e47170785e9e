"""set_state from device arrays that are freed right after it: their memory may belong to another
stream than the handle's and be handed out again there while the copies are still queued behind
earlier steps.  The state that arrives is the one that was passed."""
import numpy as np
import pytest

from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


def _arrays(n, seed):
    rng = np.random.default_rng(seed)
    return [rng.normal(size=k).astype(np.float32) for k in (3 * n + 3, 3 * n + 3, 4 * n, 3 * n)]


def _busy(b):
    """Some milliseconds of steps on the handle's stream."""
    b.step(1500, 1500)


def _reuse(arrays, stream):
    """Takes freed memory of these sizes again on the stream and overwrites it."""
    import torch
    with torch.cuda.stream(stream):
        for _ in range(3):
            for a in arrays:
                torch.full((a.size,), 9.0, device="cuda")


@pytest.mark.parametrize("made_on", ["default", "other", "handle"])
@pytest.mark.parametrize("called_on", ["handle", "default", "another"])
@pytest.mark.parametrize("handle_on", ["own", "default"])
def test_arrays_freed_right_after(handle_on, made_on, called_on):
    import torch
    n = 600
    handle = torch.cuda.Stream() if handle_on == "own" else torch.cuda.default_stream()
    made = {"default": torch.cuda.default_stream(), "other": torch.cuda.Stream(), "handle": handle}[made_on]
    call = {"default": torch.cuda.default_stream(), "another": torch.cuda.Stream(), "handle": handle}[called_on]
    spec, st = W.straight_rod(n, dt=1e-6)
    b = R.RodBatch([spec], handle.cuda_stream)
    b.set_tuning(4, 4, 10)
    for seed in range(3):
        b.set_state_rods([st])
        want = _arrays(n, seed)
        with torch.cuda.stream(made):
            dev = [torch.from_numpy(a).cuda() for a in want]
        torch.cuda.synchronize()
        _busy(b)
        with torch.cuda.stream(call):
            b.set_state(*dev)
        del dev
        _reuse(want, made)
        assert all(np.array_equal(u, v) for u, v in zip(want, b.get_state()))
    b.close()


def test_rollout_inputs_freed_right_after():
    """The initial state of a rollout, made on the default stream, dropped while the rollout's
    copies wait on the handle's stream."""
    import torch
    n = 100
    s = torch.cuda.Stream()
    spec, st = W.straight_rod(n, dt=1e-6)
    b = R.RodBatch([spec], s.cuda_stream)
    fn = R.rollout_function()
    state = [np.ascontiguousarray(a, np.float32).reshape(-1) for a in (st.x, st.v, st.q, st.w)]
    tips = []
    for busy in (False, True):
        b.set_state_rods([st])
        m = torch.ones(1, device="cuda")
        dev = [torch.from_numpy(a).cuda() for a in state]
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            if busy:
                _busy(b)
            t = fn.apply(b, m, m, *dev, 20, 5)
        del dev
        _reuse(state, torch.cuda.default_stream())
        torch.cuda.synchronize()
        tips.append(t.cpu().numpy())
    b.close()
    assert np.array_equal(*tips)
