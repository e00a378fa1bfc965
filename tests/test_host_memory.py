"""Calls that run out of device memory report it and leave a handle that later
calls can use: no launch gets a null pointer in place of a buffer."""
import pytest

from tests.host_lib import ENOMEM, OK, host_lib


@pytest.fixture
def host(tmp_path_factory):
    h = host_lib(tmp_path_factory)
    yield h
    h.lib.stub_malloc_countdown(-1)


@pytest.mark.parametrize("nth", [0, 1])
def test_wilson_buffers(host, nth):
    """The nth of the buffers that a larger call needs cannot be had: the
    smaller call that fitted before allocates its own again."""
    h = host.create((4, 4, 4, 32))
    assert host.wilson(h, 2, 4) == OK
    host.lib.stub_malloc_countdown(nth)
    assert host.wilson(h, 4, 32) == ENOMEM
    host.lib.stub_clear()
    for R, T in ((2, 4), (4, 32)):
        assert host.wilson(h, R, T) == OK
        assert host.names() and host.lib.stub_nulls() == 0
    assert host.lib.su2_destroy(h) == OK


@pytest.mark.parametrize("nth", [0, 1])
def test_smeared_buffers(host, nth):
    h = host.create((4, 4, 4, 8))
    host.lib.stub_malloc_countdown(nth)
    assert host.lib.su2_ape_smear(h, 0.5, 2) == ENOMEM
    host.lib.stub_clear()
    assert host.lib.su2_ape_smear(h, 0.5, 2) == OK and host.wilson(h, 2, 2) == OK
    assert host.names() and host.lib.stub_nulls() == 0
    assert host.lib.su2_destroy(h) == OK
