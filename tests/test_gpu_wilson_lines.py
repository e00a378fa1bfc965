"""Wilson loops against the oracle where their work split has edges: lines
longer than a workgroup holds, tiles beyond 32 sites, several time pieces,
times beyond 16, line groups that do not divide, and links off the group.
Tolerances as for the other Wilson-loop parity tests: 1e-13 in binary64,
2e-5 in binary32 (2(R+T) binary32 products at most)."""
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
    ((300, 2, 2, 4), 2, 3),    # a line longer than a workgroup: pieces with a halo
    ((2, 2, 700, 2), 2, 2),    # the same along z
    ((34, 4, 36, 6), 4, 6),    # tiles of 32 with a remainder, in both planes
    ((6, 10, 4, 22), 4, 17),   # one time in the second pass
    ((4, 6, 2, 70), 2, 32),    # time pieces, two full passes
    ((10, 14, 6, 10), 6, 10),  # line groups and time pieces that do not divide
    ((2, 2, 2, 2), 1, 1),
    ((16, 16, 16, 4), 16, 4),  # R = N: the line closes on itself
])
def test_work_split_edges(su2, orc, dims, Rm, Tm):
    U = inputs.random_config(dims, 61)
    U32 = U.astype(np.float32).astype(np.float64)
    for prec, ref, tol in ((su2.F64, U, 1e-13), (su2.F32, U32, 2e-5)):
        lat = su2.Lattice(dims, start=su2.COLD, prec=prec)
        lat.set_links(ref)
        W = lat.wilson_loops(Rm, Tm)
        assert np.abs(W - orc.wilson(dims, ref, Rm, Tm)).max() < tol, prec
        lat.ape_smear(0.6, 2)
        S = orc.ape(dims, ref, 0.6, 2)
        assert np.abs(lat.wilson_loops(Rm, Tm) - orc.wilson(dims, ref, Rm, Tm, S)).max() < tol, prec
        lat.close()


def test_links_off_the_group(su2, orc):
    """Links of norm 1 +- 4e-7, which set_links accepts: the loop is the trace
    of the links' own products, norms included."""
    dims = (4, 6, 4, 8)
    U = inputs.random_config(dims, 62)
    U *= 1.0 + 4e-7 * np.random.default_rng(63).uniform(-1.0, 1.0, U.shape[:2])[:, :, None]
    lat = su2.Lattice(dims, start=su2.COLD, prec=su2.F64)
    lat.set_links(U)
    assert np.abs(lat.wilson_loops(4, 8) - orc.wilson(dims, U, 4, 8)).max() < 1e-13
    lat.close()


@pytest.mark.parametrize("dims,Rm,Tm", [((64, 64, 64, 32), 64, 32), ((82, 82, 82, 12), 82, 12)])
def test_long_lines_take_fewer_times_at_once(su2, dims, Rm, Tm):
    """Binary64 bounds whose sums and lines do not fit the LDS at sixteen times
    a pass: the same values as calls of fewer R, or of fewer T, which fit."""
    lat = su2.Lattice(dims, start=su2.HOT, seed=64, prec=su2.F64)
    lat.ape_smear(0.6, 5)
    W = np.asarray(lat.wilson_loops(Rm, Tm))
    assert np.isfinite(W).all() and W.shape == (Rm, Tm)
    for R, T in ((Rm // 2, Tm), (Rm, 4)):
        assert np.abs(W[:R, :T] - np.asarray(lat.wilson_loops(R, T))).max() < 1e-13, (R, T)
    lat.close()


def test_more_times_than_grid_rows(su2, orc):
    """Nt + Tmax beyond 8 x 4096 times, the rows of one grid."""
    dims = (2, 2, 4, 32780)
    U = inputs.random_config(dims, 65)
    lat = su2.Lattice(dims, start=su2.COLD, prec=su2.F64)
    lat.set_links(U)
    assert np.abs(lat.wilson_loops(2, 3) - orc.wilson(dims, U, 2, 3)).max() < 1e-13
    lat.close()
