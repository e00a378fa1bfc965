"""What the library's host code launches, followed on the CPU over a stub of the
HIP runtime."""
import pytest

from tests.host_lib import F32, F64, OK, host_lib


@pytest.fixture
def host(tmp_path_factory):
    return host_lib(tmp_path_factory)


def test_lds_limits_do_not_depend_on_the_call(host):
    """A kernel's dynamic LDS limit is shared by all handles and threads: calls
    of different sizes set the same one."""
    for prec in (F32, F64):
        for dims in ((6, 4, 4, 8), (8, 4, 4, 8)):      # 96 and 128 KiB in binary64
            h = host.create(dims, prec)
            assert host.lib.su2_overrelax(h, 1) == OK
            assert host.lib.su2_destroy(h) == OK
    h = host.create((82, 82, 82, 12), F64)             # lines that take more than 64 KiB
    assert host.wilson(h, 80, 12) == OK and host.wilson(h, 82, 8) == OK
    assert host.lib.su2_destroy(h) == OK
    assert host.lib.stub_attrs() >= 2 and host.lib.stub_attr_changes() == 0
