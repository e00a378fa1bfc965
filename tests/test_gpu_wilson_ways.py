"""Wilson loops in the temporal gauge on the edges of its work split, at bounds
that go that way, and the two ways against each other.  Against the oracle:
1e-13 in binary64, 2e-5 in binary32, as for the other Wilson-loop tests."""
import numpy as np
import pytest

from tests import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def su2():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1010_4834_amd import su2 as s
    return s


@pytest.mark.parametrize("dims,Rm,Tm", [
    ((300, 2, 2, 16), 2, 12),  # a line longer than a workgroup: pieces with a halo
    ((4, 4, 300, 32), 4, 16),  # the same along z
    ((34, 4, 36, 16), 4, 16),  # tiles of 32 with a remainder, in both planes
    ((10, 14, 6, 12), 6, 12),  # line groups and time pieces that do not divide
    ((2, 2, 2, 16), 2, 8),
    ((16, 16, 16, 8), 16, 8),  # R = N: the line closes on itself
])
def test_gauge_edges(su2, orc, dims, Rm, Tm):
    U = inputs.random_config(dims, 91)
    U32 = U.astype(np.float32).astype(np.float64)
    for prec, ref, tol in ((su2.F64, U, 1e-13), (su2.F32, U32, 2e-5)):
        lat = su2.Lattice(dims, start=su2.COLD, prec=prec)
        lat.set_links(ref)
        assert np.abs(lat.wilson_loops(Rm, Tm) - orc.wilson(dims, ref, Rm, Tm)).max() < tol, prec
        lat.close()


@pytest.mark.parametrize("dims,R,T,r,t", [
    ((24, 24, 24, 24), 4, 8, 1, 1),
    ((48, 48, 48, 4), 12, 4, 2, 2),
    ((8, 8, 8, 32780), 8, 16, 1, 2),   # Nt + Tmax beyond 8 x 4096 times, the rows of one grid
])
def test_ways_agree(su2, dims, R, T, r, t):
    """The larger bounds go through the gauge, the smaller ones by transport."""
    for prec, tol in ((su2.F64, 1e-13), (su2.F32, 2e-5)):
        lat = su2.Lattice(dims, start=su2.HOT, seed=92, prec=prec)
        if dims[3] < 1000:
            lat.ape_smear(0.6, 5)
        W = np.asarray(lat.wilson_loops(R, T))
        assert np.abs(W[:r, :t] - np.asarray(lat.wilson_loops(r, t))).max() < tol, prec
        lat.close()
