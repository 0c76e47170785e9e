"""rollout_function() takes the two multipliers in whatever form set_stiffness_mult does: shapes,
types and devices of their own; a wrong number of them is refused."""
import numpy as np
import pytest

from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["plain", "columns", "twist column", "twist on the host", "double",
                                  "mixed types", "strided"])
def test_forms_of_the_multipliers(form):
    import torch
    rods = [W.straight_rod(n, dt=1e-6) for n in (20, 30, 25)]
    b = R.RodBatch([s for s, _ in rods])
    fn = R.rollout_function()
    state = [torch.from_numpy(np.concatenate([np.asarray(getattr(st, k), np.float32).reshape(-1)
                                              for _, st in rods])).cuda() for k in "xvqw"]
    bend = torch.tensor([0.8, 1.0, 1.25], device="cuda")
    twist = torch.tensor([1.1, 0.9, 1.5], device="cuda")
    want = fn.apply(b, bend, twist, *state, 12, 4)
    if form == "columns":
        bend, twist = bend[:, None], twist[:, None]
    elif form == "twist column":
        twist = twist[:, None]
    elif form == "twist on the host":
        twist = twist.cpu()
    elif form == "double":
        bend, twist = bend.double(), twist.double()
    elif form == "mixed types":
        bend = bend.double()
    elif form == "strided":
        twist = torch.stack((twist, bend), 1)[:, 0]
    got = fn.apply(b, bend, twist, *state, 12, 4)
    b.set_stiffness_mult(bend.cpu().numpy(), twist.cpu().numpy())
    assert torch.equal(want, got)
    with pytest.raises(ValueError):
        fn.apply(b, bend, twist.reshape(-1)[:2], *state, 12, 4)
    b.close()
