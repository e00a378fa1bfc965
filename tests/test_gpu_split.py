"""Heat-bath substeps with four lanes per link (lattices up to split_sites
sites) against the single-lane substeps, which two links per lane select:
links, try counts and sweep counter bit for bit, for both samplers, partial
workgroups, several lattices and every number of wavefronts per tile; the
fused plaquette up to the rounding of its sum (1e-14)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def su2():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1010_4834_amd import su2 as s
    return s


@pytest.mark.parametrize("sampler", ["HYBRID", "CREUTZ"])
@pytest.mark.parametrize("prec", ["F32", "F64"])
@pytest.mark.parametrize("dims,block", [
    ([(6, 10, 6, 4)], 256),                       # 720 links: the last workgroup partly filled
    ([(10, 6, 14, 18)], 64),
    ([(8, 6, 4, 10), (2, 2, 2, 2), (12, 8, 8, 6)], 192),
    ([(16, 16, 16, 8)], 128),                     # the largest binary64 Kennedy-Pendleton lattice
    ([(16, 16, 16, 8)], 256),
])
def test_four_lanes_per_link(su2, dims, block, prec, sampler):
    betas = [0.5 + 0.9 * i for i in range(len(dims))]   # both branches of the hybrid sampler
    got = []
    for nl in (1, 2):
        ens = su2.Ensemble(dims, betas, start=su2.HOT, seed=31, prec=getattr(su2, prec))
        su2.su2_ensemble_set_launch(ens.h, block, 0, 1, nl)
        su2.su2_ensemble_set_sampler(ens.h, getattr(su2, sampler))
        series = [ens.run(n, 31, measure_every=e) for n, e in ((5, 1), (1, 1), (4, 2))]
        got.append((series, [ens.get_links(i) for i in range(len(dims))], ens.stats()))
        ens.close()
    a, b = got
    for (p, q), (p2, q2) in zip(a[0], b[0]):
        assert np.abs(p - p2).max() < 1e-14 and np.abs(q - q2).max() < 1e-14
    assert all(np.array_equal(x, y) for x, y in zip(a[1], b[1]))
    assert a[2] == b[2]


def test_nonfinite_staples_counted(su2):
    """A NaN link makes the same links NaN with four lanes per link as with
    one, and the sweep reports it once."""
    import torch
    got = []
    for nl in (1, 2):
        lat = su2.Lattice((8, 6, 8, 10), start=su2.HOT, seed=3, prec=su2.F64)
        su2.su2_set_launch(lat.h, 128, 0, 1, nl)
        lat._buf.view(torch.float64).view(8, -1)[6, 40:44] = float("nan")
        torch.cuda.synchronize()
        with pytest.raises(su2.SU2Error) as e:
            lat.substep(2.3, 3, 0, 0)
            lat.stats()
        assert e.value.status == su2.ENUMERIC
        lat.stats()
        got.append(lat.get_links())
        lat.close()
    assert np.array_equal(got[0], got[1], equal_nan=True) and np.isnan(got[0]).any()
