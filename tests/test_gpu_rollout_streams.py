"""rollout_function() on a handle whose stream is not torch's current one: the initial state and the
gradient of the tips may still be in the making on the current stream when they are passed."""
import numpy as np
import pytest

from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


def _later(t):
    """A tensor equal to t, ready only after some milliseconds of the current stream's work."""
    import torch
    a = torch.full((4096, 4096), 1e-4, device="cuda")
    for _ in range(20):
        a = a @ a
    out = torch.full_like(t, 3.0)
    out.copy_(t + 0.0 * a.sum())
    return out


@pytest.mark.parametrize("every", [1, 5])
def test_inputs_in_the_making(every):
    import torch
    torch.cuda.init()
    spec, st = W.straight_rod(60, dt=1e-6)
    own = torch.cuda.Stream()
    fn = R.rollout_function()
    state = [torch.from_numpy(np.ascontiguousarray(a, np.float32).reshape(-1)).cuda()
             for a in (st.x, st.v, st.q, st.w)]
    mult = torch.ones(1)
    ct = torch.randn(1, 15, 3, generator=torch.Generator().manual_seed(1)).cuda()
    results = []
    for handle, late in ((torch.cuda.default_stream(), False), (own, True)):
        b = R.RodBatch([spec], handle.cuda_stream)
        leaves = [a.clone().requires_grad_() for a in state]
        torch.cuda.synchronize()
        ins = [_later(a) for a in leaves] if late else leaves
        tips = fn.apply(b, mult, mult, *ins, 15, every)
        grads = torch.autograd.grad(tips, ins, _later(ct) if late else ct)
        torch.cuda.synchronize()
        results.append([tips.detach(), *grads])
        b.close()
    assert all(torch.equal(u, v) for u, v in zip(*results))
