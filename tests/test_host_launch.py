"""What the library's host code launches, followed on the CPU over a stub of the
HIP runtime."""
import ctypes as C
import time

import pytest

from tests.host_lib import CREUTZ, ENOMEM, F32, F64, HYBRID, OK, host_lib


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


def wilson_kernels(host, dims, prec, R, T, limit=-1):
    """Kernels of one call, as (name, number of times): 'wloops4' takes up to 4
    times at once, 'wtrace' is the other way."""
    h = host.create(dims, prec)
    host.lib.stub_clear()
    host.lib.stub_malloc_limit(limit)
    st = host.wilson(h, R, T)
    host.lib.stub_malloc_limit(-1)
    assert host.lib.stub_nulls() == 0 and host.lib.su2_destroy(h) == OK
    names = ["wloops" + n.split("wloopsI")[1].split("Li")[1].split("E")[0] if "wloops" in n else
             "wtrace" if "wtrace" in n else n for n in host.names() if "wloops" in n or "wtrace" in n]
    return st, sorted((n, names.count(n)) for n in set(names))


@pytest.mark.parametrize("dims,R,T,f64,f32", [
    ((24, 24, 24, 48), 12, 16, "wloops16", "wloops16"),
    ((24, 24, 24, 48), 4, 4, "wloops4", "wloops4"),
    ((24, 24, 24, 48), 1, 1, "wtrace", "wtrace"),       # few (R, T): the rotation costs more than it saves
    ((64, 64, 64, 16), 1, 16, "wloops16", "wtrace"),
    ((4, 4, 4, 2048), 4, 16, "wtrace", "wtrace"),       # few sites over many times
    ((8, 8, 8, 12), 4, 6, "wloops8", "wloops8"),
    ((2, 2, 2, 2), 1, 1, "wtrace", "wtrace"),
])
def test_wilson_ways(host, dims, R, T, f64, f32):
    for prec, kernel in ((F64, f64), (F32, f32)):
        assert wilson_kernels(host, dims, prec, R, T) == (OK, [(kernel, 1)])


@pytest.mark.parametrize("dims,R,T,limit,kernel", [
    ((24, 24, 24, 48), 2, 8, 66 << 20, "wtrace"),   # 71 MB of rotated links, 64 MB of lines
    ((48, 48, 48, 4), 4, 1, 60 << 20, "wloops4"),   # 85 MB of lines, 51 MB of rotated links
])
def test_wilson_other_way_without_memory(host, dims, R, T, limit, kernel):
    st, names = wilson_kernels(host, dims, F32, R, T)
    assert st == OK and names != [(kernel, 1)]
    assert wilson_kernels(host, dims, F32, R, T, limit) == (OK, [(kernel, 1)])
    assert wilson_kernels(host, dims, F32, R, T, 1 << 20)[0] == ENOMEM


@pytest.mark.parametrize("n,nt,T,prec,kernels", [
    (80, 32, 32, F64, [("wloops16", 2)]),
    (82, 12, 12, F64, [("wloops4", 1), ("wloops8", 1)]),
    (138, 16, 16, F64, [("wloops4", 4)]),
    (110, 16, 16, F32, [("wloops16", 1)]),
    (112, 16, 16, F32, [("wloops8", 2)]),
])
def test_long_lines_take_fewer_times(host, n, nt, T, prec, kernels):
    """Rmax = n: the sums of sixteen times leave no room for the lines."""
    assert wilson_kernels(host, (n, n, n, nt), prec, n, T) == (OK, kernels)


def test_wilson_first_call_allocates_no_host_memory(host):
    before = host.lib.stub_host_mallocs()
    h = host.create((8, 8, 8, 12))
    n = host.lib.stub_host_mallocs()
    assert n == before + 1     # results and state words of a handle together
    assert host.wilson(h, 4, 6) == OK and host.wilson(h, 8, 12) == OK and host.lib.stub_host_mallocs() == n
    assert host.lib.su2_destroy(h) == OK


@pytest.mark.parametrize("dims", [(8, 8, 8, 48), (16, 16, 16, 512)])
def test_wilson_bounds_in_turn(host, dims):
    """A program that alternates between two bounds pays for no new work split on
    each call (searched anew, 10 to 100 times the rest of a call's host work here)."""
    h = host.create(dims)

    def fastest(bounds):
        best = 1.0
        for _ in range(30):
            t = time.perf_counter()
            for _ in range(10):
                for b in bounds:
                    host.wilson(h, *b)
            best = min(best, time.perf_counter() - t)
        host.lib.stub_clear()
        return best

    same = fastest([(8, 16), (8, 16)])
    assert fastest([(8, 16), (8, 15)]) < 3 * same
    assert host.lib.su2_destroy(h) == OK


@pytest.mark.parametrize("dims,steps,f64,f32", [
    ((2, 2, 2, 512), 25, True, True),
    ((2, 2, 2, 514), 25, False, False),    # idle lanes: one launch per step
    ((4, 4, 2, 2048), 2, True, False),
    ((4, 4, 2, 2050), 4, False, False),
    ((4, 4, 2, 4096), 5, True, True),
    ((4, 4, 2, 4098), 5, False, False),
    ((4, 2, 2, 65536), 5, False, False),
    ((6, 4, 2, 65536), 3, True, True),
    ((4, 4, 4, 4), 2, True, True),
    ((4, 4, 4, 4), 1, False, False),
    ((6, 4, 4, 64), 2, True, False),       # a quarter of the lanes idle
    ((6, 6, 6, 64), 2, True, True),
    ((8, 8, 4, 64), 2, True, True),
    ((8, 8, 8, 64), 4, True, False),       # large slices
    ((8, 8, 8, 64), 5, True, True),
    ((16, 8, 8, 4), 5, False, True),
    ((16, 8, 10, 4), 25, False, False),
])
def test_smearing_ways(host, dims, steps, f64, f32):
    for prec, slices in ((F64, f64), (F32, f32)):
        h = host.create(dims, prec)
        host.lib.stub_clear()
        assert host.lib.su2_ape_smear(h, 0.5, steps) == OK
        names = host.names()
        assert len(names) == (1 if slices else steps) and all(("k_ape_slices" in n) == slices for n in names), prec
        assert host.lib.su2_destroy(h) == OK


@pytest.mark.parametrize("dims,f64,f32", [
    ((64, 64, 64, 64), 0, 0),
    ((64, 64, 64, 8), 1, 0),
    ((64, 64, 64, 12), 1, 0),
    ((64, 64, 64, 14), 0, 0),
    ((64, 64, 128, 12), 0, 1),
    ((64, 64, 128, 14), 0, 0),
    ((96, 64, 128, 8), 1, 1),      # one time slice per XCD: 30% slower in round robin
    ((128, 128, 64, 8), 1, 1),
    ((32, 32, 32, 32), 3, 3),
    ((80, 80, 80, 16), 1, 3),      # large slices over few times
    ((112, 112, 112, 8), 1, 1),
    ((64, 64, 8, 128), 1, 1),
    ((20, 24, 24, 48), 1, 1),      # small slices
    ((24, 24, 32, 32), 3, 3),
    ((26, 26, 32, 40), 1, 1),
    ((34, 34, 32, 32), 3, 3),
    ((24, 24, 24, 32), 1, 1),
])
def test_tile_mode_of_a_new_lattice(host, dims, f64, f32):
    for prec, mode in ((F64, f64), (F32, f32)):
        h = host.create(dims, prec)
        assert host.launch(h) == (256, 0, mode, 1)
        assert host.lib.su2_destroy(h) == OK


def launches(host, what):
    host.lib.stub_clear()
    assert what() == OK
    return [(n, host.lib.stub_xcd(i), host.lib.stub_tiles(i)) for i, n in enumerate(host.names())]


@pytest.mark.parametrize("dims,prec,walk", [((64, 64, 64, 16), F32, 0), ((64, 64, 64, 16), F64, 1),
                                            ((128, 128, 64, 16), F32, 1)])
def test_measurements_of_a_round_robin_lattice(host, dims, prec, walk):
    """The tile mode chosen for the heat bath is not the plaquette's everywhere,
    and never the Polyakov loop's; a mode that the caller sets is both's."""
    h = host.create(dims, prec)
    assert host.launch(h)[2] == 0
    out = (C.c_double * 1)()
    for mode, want in ((None, (walk, 1)), (0, (0, 0)), (1, (1, 1))):
        if mode is not None:
            assert host.lib.su2_set_launch(h, 256, 0, mode, 1) == OK
        seen = {n.split("k_")[1][:4]: x for n, x, _ in launches(host, lambda: host.plaquette(h)) +
                launches(host, lambda: host.lib.su2_polyakov(h, out))}
        assert (seen["plaq"], seen["poly"]) == want, mode
    assert host.lib.su2_destroy(h) == OK


@pytest.mark.parametrize("dims,same", [((32, 32, 32, 32), True), ((20, 24, 24, 48), False)])
def test_overrelaxation_tiles_in_mode_3(host, dims, same):
    """Over-relaxation takes the heat bath's blocks on lattices they suit only
    (20 x 24^2 x 48: 10.2 us a substep, 8.8 in lexicographic order)."""
    h = host.create(dims)
    assert host.lib.su2_set_launch(h, 256, 0, 3, 1) == OK
    over = [t for n, _, t in launches(host, lambda: host.lib.su2_overrelax(h, 1)) if "overrelax" in n]
    heat = [t for n, _, t in launches(host, lambda: host.lib.su2_heatbath(h, 2.3, 1, 1)) if "heatbath" in n]
    assert len(over) == len(heat) == 8 and (over == heat) == same
    assert host.lib.su2_destroy(h) == OK


@pytest.mark.parametrize("dims,prec,sampler,beta,four", [
    ((16, 16, 16, 16), F32, CREUTZ, 0.0, True),
    ((16, 16, 16, 20), F32, CREUTZ, 0.0, False),   # one try is most links' last
    ((16, 16, 16, 24), F32, CREUTZ, 0.2, True),
    ((16, 16, 16, 32), F32, CREUTZ, 0.2, False),
    ((16, 16, 16, 32), F32, CREUTZ, 1.0, True),
    ((16, 16, 16, 34), F32, CREUTZ, 6.0, False),
    ((16, 16, 16, 8), F64, CREUTZ, 0.0, True),
    ((16, 16, 16, 16), F64, CREUTZ, 0.0, False),
    ((16, 16, 16, 16), F64, CREUTZ, 1.0, True),
    ((16, 16, 16, 24), F64, CREUTZ, 1.0, False),
    ((16, 16, 16, 24), F64, CREUTZ, 2.0, True),
    ((16, 16, 16, 8), F64, HYBRID, 0.0, False),
    ((16, 16, 16, 8), F64, HYBRID, 0.3, True),
    ((16, 16, 16, 10), F64, HYBRID, 2.3, False),
    ((8, 8, 8, 8), F32, HYBRID, 2.3, False),
])
def test_four_lanes_per_link(host, dims, prec, sampler, beta, four):
    """By size, sampler, precision and coupling, also in a graph that was captured
    at another coupling."""
    h = host.create(dims, prec)
    assert host.lib.su2_set_sampler(h, sampler) == OK
    for b in (2.3, beta):
        assert host.lib.su2_heatbath(h, b, 2, 1) == OK
    host.lib.stub_clear()
    assert host.lib.su2_heatbath_substep(h, beta, 1, 0, 0) == OK
    names = host.names()
    assert len(names) == 1 and ("k_heatbath_split" in names[0]) == four
    host.lib.stub_clear()
    assert host.lib.su2_heatbath(h, 2.3, 2, 1) == OK and host.lib.su2_heatbath(h, beta, 2, 1) == OK
    now = [n for n in host.names() if "k_heatbath" in n]
    assert not now or ("split" in now[-1]) == four     # captured anew where the kernel is another
    assert host.lib.su2_destroy(h) == OK


def test_tuned_shape_is_of_the_same_lattice_and_sampler(host):
    """The shapes that the tuner keeps for later handles."""
    def tuned(dims, prec=F64, sampler=HYBRID, beta=2.3):
        h = host.create(dims, prec)
        assert host.lib.su2_set_sampler(h, sampler) == OK
        host.lib.stub_clear()
        assert host.lib.su2_autotune(h, beta) == OK
        trials = sum("k_heatbath" in n for n in host.names())
        assert host.lib.su2_destroy(h) == OK
        return trials > 0

    assert tuned((10, 12, 14, 16)) and not tuned((10, 12, 14, 16)) and not tuned((10, 12, 14, 16), beta=2.4)
    assert tuned((10, 12, 14, 16), sampler=CREUTZ) and not tuned((10, 12, 14, 16), sampler=CREUTZ)
    assert tuned((14, 12, 10, 16)) and tuned((10, 14, 12, 16))   # as many sites, the same Nt
    assert tuned((10, 12, 14, 16), prec=F32)


@pytest.mark.parametrize("dims,f64,f32", [
    ((4, 4, 4, 4), 1, 1),
    ((2, 2, 2, 64), 1, 1),
    ((2, 2, 2, 66), 2, 1),       # one tile
    ((4, 4, 4, 4096), 2, 1),
    ((8, 8, 8, 24), 1, 1),
    ((8, 8, 8, 26), 2, 1),       # two tiles, one after the other in one launch
    ((8, 8, 8, 64), 2, 1),
    ((8, 8, 8, 66), 2, 2),
    ((8, 8, 10, 4), 2, 2),       # three tiles
])
def test_polyakov_launches(host, dims, f64, f32):
    for prec, n in ((F64, f64), (F32, f32)):
        h = host.create(dims, prec)
        host.lib.stub_clear()
        assert host.lib.su2_polyakov(h, (C.c_double * 1)()) == OK
        assert len(host.names()) == n
        assert host.lib.su2_destroy(h) == OK
