"""The counters by which chunks wait on each other: their order across the ends of the signed and
the unsigned 32-bit range (a step count compared as a signed number let a wait pass at once after
2^31 steps), and how far a launch raises them."""
import os

import pytest

import host_stub


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    if not os.path.exists(host_stub.HIPCC):
        pytest.skip("needs hipcc")
    return host_stub.Stub(host_stub.build(str(tmp_path_factory.mktemp("stub")))).lib


@pytest.mark.parametrize("at", [0, 1, 2**31 - 2, 2**31 - 1, 2**31, 2**31 + 1, 2**32 - 2, 2**32 - 1])
def test_order_holds_across_the_range(L, at):
    for ahead in range(1, 5):
        later = (at + ahead) % 2**32
        assert L.chunk_mark_behind(at, later) == 1
        assert L.chunk_mark_behind(later, at) == 0
    assert L.chunk_mark_behind(at, at) == 0


def test_handles_start_just_below_the_signed_limit(L):
    assert 0 < 2**31 - L.chunk_first_mark() <= 16


@pytest.mark.parametrize("every", [1, 2, 5, 16])
def test_marks_of_a_launch_are_its_load_and_exchanges(L, every):
    for n in range(1, 60):   # an exchange after every `every` steps but the last step
        assert L.chunk_launch_marks(n, every) == 1 + sum((s + 1) % every == 0 and s + 1 != n
                                                         for s in range(n))
