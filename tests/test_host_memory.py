"""Calls that run out of device memory report it and leave a handle that later
calls can use: no launch gets a null pointer in place of a buffer."""
import pytest

from tests.host_lib import ENOMEM, ESTATE, OK, host_lib


@pytest.fixture
def host(tmp_path_factory):
    h = host_lib(tmp_path_factory)
    yield h
    h.lib.stub_malloc_countdown(-1)
    h.lib.stub_malloc_limit(-1)
    h.lib.stub_malloc_room(-1)


@pytest.mark.parametrize("room", [0, 1])
def test_wilson_buffers(host, room):
    """The first or the second of the buffers that a larger call needs cannot be
    had: the smaller call that fitted before allocates its own again."""
    h = host.create((4, 4, 4, 32))
    assert host.wilson(h, 2, 4) == OK
    host.lib.stub_malloc_room(room)
    assert host.wilson(h, 4, 32) == ENOMEM
    host.lib.stub_malloc_room(-1)
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


def sweep(host, h):
    """Every kind of launch that reads the tables."""
    host.lib.stub_clear()
    assert host.lib.su2_heatbath(h, 2.3, 3, 1) == OK and host.lib.su2_overrelax(h, 1) == OK
    assert host.plaquette(h) == OK and host.lib.su2_ape_smear(h, 0.5, 1) == OK
    assert host.names() and host.lib.stub_nulls() == 0


def test_launch_shape(host):
    """A launch shape one of whose tables, each in turn, cannot be had is
    refused, and the old one stays."""
    st, nth = ENOMEM, 0
    while st != OK:
        h = host.create((8, 8, 8, 8))
        shape = host.launch(h)
        host.lib.stub_malloc_countdown(nth)
        st = host.lib.su2_set_launch(h, 64, 512, 1, 2)
        host.lib.stub_malloc_countdown(-1)
        assert st in (ENOMEM, OK)
        assert host.launch(h) == (shape if st else (64, 512, 1, 2))
        sweep(host, h)
        assert host.lib.su2_destroy(h) == OK
        nth += 1
    assert nth > 10


def test_launch_shape_without_any(host):
    """Neither the new shape's tables nor the old one's: the handle is failed."""
    h = host.create((8, 8, 8, 8))
    host.lib.stub_malloc_limit(0)
    assert host.lib.su2_set_launch(h, 64, 0, 1, 1) == ENOMEM
    host.lib.stub_malloc_limit(-1)
    assert host.lib.su2_heatbath(h, 2.3, 1, 1) == ESTATE and host.plaquette(h) == ESTATE
    assert host.lib.su2_destroy(h) == OK


@pytest.mark.parametrize("nth", [1, 5, 60])
def test_autotune(host, nth):
    """A candidate without room for its tables is passed over."""
    h = host.create((8, 8, 8, 8 + 2 * nth))   # a size of its own: nothing is tuned yet
    host.lib.stub_malloc_countdown(nth)
    assert host.lib.su2_autotune(h, 2.3) == OK
    sweep(host, h)
    assert host.lib.su2_destroy(h) == OK
