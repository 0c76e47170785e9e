"""A handle that reported a condition (a non-finite state, too many contacts, a non-finite adjoint)
is whole again after the next set_state: the condition is latched until then and no longer."""
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


def _fails(call, status):
    with pytest.raises(R.RodError) as e:
        call()
    assert R.STATUS[e.value.status] == status


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("n", [64, 500, 3000])
def test_after_a_non_finite_state(n, device):
    import torch
    spec, st = W.straight_rod(n, dt=1e-7)
    bad = W.RodState(st.x.copy(), st.v, st.q, st.w)
    bad.x[n // 2] = np.nan
    b = R.RodBatch([spec])

    def put(s):
        a = [np.ascontiguousarray(k, np.float32).reshape(-1) for k in (s.x, s.v, s.q, s.w)]
        b.set_state(*([torch.from_numpy(k).cuda() for k in a] if device else a))

    put(st)
    b.step(20, 10)
    b.sync()
    want = b.get_state()
    put(bad)
    b.step(5, 5)
    for _ in range(2):
        _fails(b.sync, "ROD_E_UNSTABLE")
    put(st)
    b.step(20, 10)
    b.sync()
    assert all(np.array_equal(u, v) for u, v in zip(want, b.get_state()))
    b.close()


def test_after_too_many_contacts():
    n = 40
    spec, st = W.straight_rod(n, L=0.04, radius=0.01, inextensible=True, dt=1e-7)
    other = W.RodState(st.x + [0.0, 0.0, 0.015], st.v, st.q, st.w)   # inside its neighbour
    apart = W.RodState(st.x + [0.0, 0.0, 0.5], st.v, st.q, st.w)
    b = R.RodBatch([spec, spec.replace(clamp_x0=(0.0, 0.0, 0.015))])
    b.set_contact([[0, 1]], 0.1)
    b.set_state_rods([st, other])
    b.step(1, 1)
    _fails(b.sync, "ROD_E_UNSUPPORTED")
    b.set_clamp(1, (0.0, 0.0, 0.5), spec.clamp_q0)
    b.set_state_rods([st, apart])
    b.step(1, 1)
    b.sync()
    b.close()


def test_after_a_non_finite_adjoint():
    spec, st = W.straight_rod(30, dt=1e-6)
    b = R.RodBatch([spec])
    ct = np.ones((1, 6, 3), np.float32)
    b.set_state_rods([st])
    b.adjoint_forward(6, 3)
    want = b.adjoint_backward(ct)
    b.set_state_rods([st])
    b.adjoint_forward(6, 3)
    _fails(lambda: b.adjoint_backward(np.full_like(ct, np.inf)), "ROD_E_UNSTABLE")
    b.set_state_rods([st])
    b.adjoint_forward(6, 3)
    got = b.adjoint_backward(ct)
    assert all(np.array_equal(want[k], got[k]) for k in want)
    b.close()
