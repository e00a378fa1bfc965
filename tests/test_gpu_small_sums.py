"""The Polyakov series of a small lattice's run against the standalone call on
the same links.  Both multiply the same links in the same order, and both sum
the sites in (hi, lo) pairs, whose total is right to far below binary64
rounding whatever the order: the values are the same bits."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def su2():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1010_4834_amd import su2 as s
    return s


@pytest.mark.parametrize("prec", ["F32", "F64"])
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (8, 4, 4, 4), (6, 4, 10, 2), (10, 8, 6, 2)])
def test_polyakov_series_is_the_standalone_value(su2, dims, prec):
    ens = su2.Ensemble([dims], [2.3], start=su2.HOT, seed=5, prec=getattr(su2, prec))
    lat = su2.Lattice(dims, start=su2.COLD, prec=getattr(su2, prec))
    for k in range(24):
        _, poly = ens.run(1, 5)
        lat.set_links(ens.get_links(0))
        assert poly[0, 0] == lat.polyakov(), k
    ens.close()
    lat.close()
