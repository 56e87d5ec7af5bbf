"""Which kernels a call launches, and what it does under capture and when memory runs out: the library's host code on a HIP
runtime without a device (tests/stub_library.py)."""
import pytest

import stub_library


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    return stub_library.link(str(tmp_path_factory.mktemp("stub")))


@pytest.fixture
def ctx(library):
    c = stub_library.StubContext(library)
    yield c
    c.close()


def test_captured_small_epochs_clear_their_own_sums(library):
    """A replay finds what the replay before it has left, not what the host counted on: a captured small epoch starts by
    clearing its sums.  Eager ones need that only where the call before has not cleared as much."""
    ctx = stub_library.StubContext(library, stream=0x1000)
    try:
        small = ["small_kernel<2,true>", "small_update_kernel"]
        assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)
        assert ctx.epoch(5000, 100, 8) == (0, small)
        ctx.capturing(True)
        for _ in range(2):
            assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)
        ctx.capturing(False)
        assert ctx.epoch(5000, 100, 8) == (0, small)
        assert ctx.epoch(5000, 49, 8) == (0, small)                                   # a smaller map
        assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)           # a larger one
        assert ctx.epoch(5000, 100, 8) == (0, small)
    finally:
        ctx.close()
