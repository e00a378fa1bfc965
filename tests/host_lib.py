"""The library's host code on the CPU: the sources compiled for the host alone
and linked with hip_stub.cpp in place of the HIP runtime."""
import ctypes as C
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1010_4834_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
OK, EINVAL, ENOMEM, ESTATE = 0, -1, -2, -5
COLD, F64, F32, HYBRID, CREUTZ = 0, 0, 1, 0, 1


def build(folder):
    objs, jobs = [], []
    for src in (os.path.join(CSRC, "su2_api.hip"), os.path.join(CSRC, "su2_kernels.hip"),
                os.path.join(HERE, "hip_stub.cpp")):
        objs.append(os.path.join(folder, os.path.basename(src) + ".o"))
        jobs.append(subprocess.Popen([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1",
                                      "-std=c++17", "-fPIC", "-I", CSRC, "-c", src, "-o", objs[-1]]))
    for j in jobs:
        assert j.wait() == 0
    # the device code that a host-only object registers is not there
    syms = subprocess.run(["nm", "-u"] + objs, capture_output=True, text=True, check=True).stdout.split()
    lib = os.path.join(folder, "libsu2_host.so")
    subprocess.run(["g++", "-shared", "-o", lib] + objs +
                   ["-Wl,--defsym=%s=0" % s for s in sorted(set(syms)) if s.startswith("__hip_fatbin")], check=True)
    return C.CDLL(lib)


_host = []


def host_lib(tmp_path_factory):
    """One build for the test session."""
    if not _host:
        _host.append(Host(tmp_path_factory.mktemp("host")))
    _host[0].lib.stub_clear()
    return _host[0]


class Host:
    """The C ABI with handles and out-parameters as Python values."""

    def __init__(self, folder):
        self.lib = build(str(folder))
        self.lib.stub_name.restype = C.c_char_p
        self.lib.stub_tiles.restype = C.c_void_p
        for f in ("limit", "countdown", "room"):
            getattr(self.lib, "stub_malloc_" + f).argtypes = [C.c_longlong]
        self.lib.su2_create.argtypes = [C.c_int] * 5 + [C.c_uint64, C.c_int, C.c_void_p, C.c_size_t, C.c_void_p]
        self.lib.su2_ensemble_run.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_uint64, C.c_void_p, C.c_void_p]
        self.lib.su2_ape_smear.argtypes = [C.c_void_p, C.c_double, C.c_int]
        self.lib.su2_heatbath.argtypes = [C.c_void_p, C.c_double, C.c_int, C.c_uint64]
        self.lib.su2_heatbath_substep.argtypes = [C.c_void_p, C.c_double, C.c_uint64, C.c_int, C.c_int]
        self.lib.su2_autotune.argtypes = [C.c_void_p, C.c_double]
        self.lib.su2_wilson_loops.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_void_p]
        for f in ("su2_destroy", "su2_release_buffers"):
            getattr(self.lib, f).argtypes = [C.c_void_p]
        for f in ("su2_overrelax", "su2_set_sampler"):
            getattr(self.lib, f).argtypes = [C.c_void_p, C.c_int]
        self.lib.su2_set_launch.argtypes = [C.c_void_p] + [C.c_int] * 4
        self.lib.su2_get_launch.argtypes = [C.c_void_p] + [C.c_void_p] * 4
        self.lib.su2_plaquette.argtypes = [C.c_void_p] * 4
        self.lib.su2_polyakov.argtypes = [C.c_void_p] * 2

    def create(self, dims, prec=F32):
        h = C.c_void_p()
        assert self.lib.su2_create(*dims, COLD, 1, prec, None, 0, C.byref(h)) == OK
        return h

    def wilson(self, h, R, T):
        return self.lib.su2_wilson_loops(h, R, T, (C.c_double * (R * T))())

    def plaquette(self, h):
        return self.lib.su2_plaquette(h, (C.c_double * 1)(), None, None)

    def launch(self, h):
        v = (C.c_int * 4)()
        at = C.addressof(v)
        assert self.lib.su2_get_launch(h, at, at + 4, at + 8, at + 12) == OK
        return tuple(v)

    def names(self):
        return [self.lib.stub_name(i).decode() for i in range(self.lib.stub_launches())]
