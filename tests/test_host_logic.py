"""What the library's host code decides, on a HIP runtime that runs no kernel (tests/hip_stub.hip):
waits, launches, captures and failed allocations."""
import ctypes as C
import os

import numpy as np
import pytest

import host_stub
from paper_2509_04277_amd import rod as R
from paper_2509_04277_amd import workloads as W

STREAM = 0x1000   # (any address: the runtime only compares them)
PER_THREAD = 2    # hipStreamPerThread


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    if not os.path.exists(host_stub.HIPCC):
        pytest.skip("needs hipcc")
    return host_stub.Stub(host_stub.build(str(tmp_path_factory.mktemp("stub"))))


@pytest.fixture
def stub(built, monkeypatch):
    monkeypatch.setattr(R, "_lib", built.lib)
    built.lib.stub_reset()
    _handles.clear()
    yield built
    for b in _handles:
        b.close()


_handles = []   # of the running test


def _handle(n, stream=STREAM, inext=True, count=1):
    """A handle of clamped rods of n elements with a state."""
    spec, st = W.straight_rod(n, dt=1e-6, inextensible=inext)
    b = R.RodBatch([spec] * count, stream)
    _handles.append(b)
    b.set_state_rods([st] * count)
    return b


def test_set_state_waits_unless_told_not_to(stub):
    b = _handle(100)
    arrays = [np.zeros(k, np.float32) for k in (303, 303, 400, 300)]
    for on_device, waits in ((0, 1), (1, 1), (R.DEVICE_QUEUED, 0)):
        before = stub.lib.stub_syncs()
        assert stub.lib.rod_set_state(b.h, *[C.c_void_p(a.ctypes.data) for a in arrays], on_device, 0.0) == 0
        assert stub.lib.stub_syncs() - before == waits


@pytest.mark.parametrize("count,inext,one_wave", [
    (500, False, False), (1200, False, False), (2048, False, False), (2049, False, True),
    (512, True, False), (513, True, True), (1200, True, True)])
def test_shape_of_many_mid_rods(stub, count, inext, one_wave):
    """Rods of 129 to 256 elements: one wavefront each from 8 wavefronts per compute unit on, in
    the shape of four; for handles without constraint iterations, which lose by it, from 32 on."""
    b = _handle(200, inext=inext, count=count)
    assert [x[:3] for x in b.buckets()] == [(1, 4, count) if one_wave else (4, 1, count)]


def test_shape_of_mixed_mid_rods(stub):
    """One bucket for extensible and inextensible rods together."""
    (e, se), (i, si) = (W.straight_rod(200, dt=1e-6, inextensible=k) for k in (False, True))
    _handles.append(R.RodBatch([e] * 400 + [i] * 400, STREAM))
    assert [x[:3] for x in _handles[0].buckets()] == [(1, 4, 800)]


def _windows(launches):
    return [l for l in launches if "rod_window_kernel" in l.kernel or "rod_grid_kernel" in l.kernel]


def test_a_captured_step_leaves_other_handles_alone(stub):
    """A handle that stepped as chunks and then steps under capture: the event that other handles'
    chunks wait for is not the one recorded in the capture."""
    a, b = _handle(2048, 0x1000), _handle(95000, 0x2000)
    a.step(10, 10)
    stub.lib.stub_capture(0x1000, 1)
    before = stub.lib.stub_launches()
    a.step(10, 10)
    assert not _windows(stub.launches(before)), "a captured step is not spread"
    stub.lib.stub_capture(0x1000, 0)
    b.step(10, 10)   # its chunks do not fit beside the other's, which are finished
    assert sum(l.grid for l in _windows(stub.launches())) > 256
    assert stub.lib.stub_waits() == 0 and stub.lib.stub_broken_captures() == 0
    a.step(10, 10)
    a.last_step_time()


def test_captured_long_rods_do_not_pass_the_gate(stub):
    a, b = _handle(65536, 0x1000), _handle(65536, 0x2000)
    a.step(10, 10)
    stub.lib.stub_hold(0x1000, 1)
    stub.lib.stub_capture(0x2000, 1)
    b.step(10, 10)
    stub.lib.stub_capture(0x2000, 0)
    stub.lib.stub_hold(0x1000, 0)
    a.step(10, 10)
    assert len(_windows(stub.launches())) == 3
    assert stub.lib.stub_waits() == 0 and stub.lib.stub_broken_captures() == 0


def test_steps_beside_a_capture_of_another_thread(stub):
    """Asking whether another handle's run is done would end a capture in the global mode."""
    hs = [_handle(2048, 0x1000 * (1 + i)) for i in range(10)]   # (room runs short: it asks)
    for h in hs[:-1]:
        h.step(10, 10)
    stub.lib.stub_strict(1)
    hs[-1].step(10, 10)
    stub.lib.stub_strict(0)
    assert stub.lib.stub_queries() > 0 and stub.lib.stub_broken_captures() == 0


def test_spread_rods_do_not_wait_for_other_handles(stub):
    """Handles of mid rods in flight on streams of their own: chunks while they fit the compute
    units together, one workgroup per rod from there on, and nothing waits."""
    hs = [_handle(2048, 0x1000 * (1 + i)) for i in range(24)]
    chunks = hs[0].chunks[0]
    fit = 128 // chunks   # half the compute units
    assert chunks > 1 and fit < len(hs)
    for i, h in enumerate(hs):
        h.step(10, 10)
        stub.lib.stub_hold(0x1000 * (1 + i), 1)
        assert h.chunks == (chunks, chunks if i < fit else 0)
        assert h.time()[1] == 10 and h.last_step_time()[1] == 1
        stub.lib.stub_hold(0x1000 * (1 + i), 1)   # (the timing waited for it)
    assert stub.lib.stub_waits() == 0
    stub.lib.stub_hold(0x1000, 0)      # the first is done: its room goes to the last
    hs[-1].step(10, 10)
    assert hs[-1].chunks == (chunks, chunks)


def test_long_rods_wait_for_what_does_not_fit_beside_them(stub):
    """Rods that step as chunks only: a run waits for every unfinished one of another stream."""
    a, b, c = (_handle(17000, 0x1000 * (1 + i)) for i in range(3))
    n = a.chunks[0]
    assert 2 * n <= 256 < 3 * n
    for i, h in enumerate((a, b, c)):
        assert stub.lib.stub_waits() == 0
        h.step(20, 10)
        stub.lib.stub_hold(0x1000 * (1 + i), 1)
    assert stub.lib.stub_waits() == 2
    a.step(20, 10)
    assert stub.lib.stub_waits() == 4
    assert all(h.chunks == (n, n) for h in (a, b, c))
    stub.lib.stub_hold(0x3000, 0)
    b.step(20, 10)      # fits beside the one that is left
    assert stub.lib.stub_waits() == 4


def test_an_earlier_larger_run_of_a_stream_counts_while_it_lasts(stub):
    """Two handles on one stream: room is taken by the larger run until it is over."""
    big, small, other = _handle(10000, 0x1000), _handle(2048, 0x1000), _handle(2000, 0x2000)
    room = 128 - big.chunks[0]
    assert room > small.chunks[0]
    more = [_handle(2048, 0x1000 * (3 + i)) for i in range(room // small.chunks[0] + 1)]
    for held in (1, 0):
        big.step(10, 10)
        stub.lib.stub_hold(0x1000, held)
        small.step(10, 10)
        stub.lib.stub_hold(0x1000, 1)
        for i, h in enumerate(more):
            h.step(10, 10)
            stub.lib.stub_hold(0x1000 * (3 + i), 1)
        other.step(10, 10)
        assert (other.chunks[1] == 0) == bool(held)
        for i in range(len(more)):
            stub.lib.stub_hold(0x1000 * (3 + i), 0)
        stub.lib.stub_hold(0x1000, 0)


def test_four_processes_of_spread_rods_fit_the_device(stub):
    """A process has at most half the compute units' number of coupled chunks in flight where the
    library chose them (the device holds two per unit), in one handle or in several; chunks that
    wait for no neighbour are not limited by this."""
    for n in (2048, 700, 400):
        each = _handle(n).chunks[0]
        assert each > 1
        for count, spread in ((128 // each, True), (128 // each + 1, False)):
            h = _handle(n, count=count)
            assert h.chunks[0] == (count * each if spread else 0)
            h.close()
    assert _handle(300, count=200).chunks[0] == 200


def test_a_spread_plan_that_does_not_fit_the_memory_leaves_no_error(stub):
    """The plan's buffers are an extra: without them rods step in one workgroup each, and the failed
    allocation is not reported by a later call."""
    plain = _handle(100)     # (how many allocations a handle makes without a plan)
    plain.close()
    before = stub.lib.stub_allocations()
    full = _handle(2048)
    made = stub.lib.stub_allocations() - before
    full.close()
    for skip in range(made - 4, made):   # the plan's four are a handle's last
        stub.lib.stub_fail_malloc(skip)
        h = _handle(2048)
        stub.lib.stub_fail_malloc(-1)
        assert h.chunks[0] == 0
        h.step(10, 10)
        h.sync()
        h.close()
    assert stub.lib.stub_allocations() == before


@pytest.mark.parametrize("spl", [10, 0])
@pytest.mark.parametrize("n", [200, 512, 2048])
@pytest.mark.parametrize("chunk_us,shape_us", [(20.0, 50.0), (50.0, 20.0)])
def test_autotune_keeps_the_faster_of_chunks_and_shapes(stub, n, spl, chunk_us, shape_us):
    h = _handle(n)
    planned = h.chunks[0]
    assert planned > 0
    stub.lib.stub_cost(b"rod_window_kernel", chunk_us)
    stub.lib.stub_cost(b"rod_resident_kernel", shape_us)
    t = h.autotune(probe_steps=10, steps_per_launch=spl)
    h.step(10, 10)
    assert (h.chunks[1] > 0) == (chunk_us < shape_us)
    ran = stub.launches()[-1].kernel
    assert ("rod_window_kernel" if chunk_us < shape_us else "rod_resident_kernel") in ran
    if h.buckets()[0][3] > 0:    # (a rod that rod_set_chunking chunks reports no time)
        assert t["us_per_step"] == pytest.approx(min(chunk_us, shape_us) / 10, rel=1e-3)
    assert h.time()[1] == 10


def test_autotune_that_fails_leaves_the_handle_as_it_was(stub):
    h = _handle(2048)
    planned = h.chunks[0]
    stub.lib.stub_fail_malloc(2)
    with pytest.raises(R.RodError):
        h.autotune(probe_steps=10)
    stub.lib.stub_fail_malloc(-1)
    stub.lib.hipGetLastError()
    assert h.chunks[0] == planned
    h.step(10, 10)
    assert h.chunks[1] == planned


def test_autotune_without_room_for_the_chunks(stub):
    """Other handles' chunks in flight: nothing to time, the handle keeps its plan for later."""
    others = [_handle(2048, 0x1000 * (2 + i)) for i in range(8)]
    for i, o in enumerate(others):
        o.step(10, 10)
        stub.lib.stub_hold(0x1000 * (2 + i), 1)
    h = _handle(2048)
    h.autotune(probe_steps=10)
    for i in range(len(others)):
        stub.lib.stub_hold(0x1000 * (2 + i), 0)
    h.step(10, 10)
    assert h.chunks[1] == h.chunks[0] > 0


def test_per_thread_streams_are_not_one_stream(stub):
    """Two handles on the per-thread stream may be stepped by two threads, side by side."""
    a, b = _handle(60000, PER_THREAD), _handle(60000, PER_THREAD)
    assert a.chunks[0] <= 256 < 2 * a.chunks[0]
    a.step(10, 10)
    stub.lib.stub_hold(PER_THREAD, 1)
    a.step(10, 10)
    assert stub.lib.stub_waits() == 0
    b.step(10, 10)
    assert stub.lib.stub_waits() == 1


def test_the_null_stream_beside_a_capture_keeps_the_order(stub):
    """The runtime does not tell the null stream's capture status while another stream captures:
    long rods are ordered as ever, mid rods step in one workgroup each."""
    a, b, c = _handle(60000, 0x2000), _handle(60000, 0), _handle(700, 0)
    a.step(10, 10)
    stub.lib.stub_hold(0x2000, 1)
    stub.lib.stub_implicit(1)
    b.step(10, 10)
    assert stub.lib.stub_waits() == 1
    c.step(10, 10)
    assert c.chunks[0] > 0 == c.chunks[1]
    stub.lib.stub_implicit(0)


def test_runs_of_other_streams_are_asked_for_only_where_room_is_short(stub):
    """What a step of a handle costs does not grow with the handles there are."""
    hs = [_handle(512, 0x1000 * (1 + i)) for i in range(40)]
    fit = 128 // hs[0].chunks[0]
    assert fit < len(hs)
    for i, h in enumerate(hs):
        h.step(10, 10)
        if i < fit:
            assert stub.lib.stub_queries() == 0
    assert stub.lib.stub_queries() > 0
    assert all(h.chunks[1] for h in hs)   # the earlier ones were over
