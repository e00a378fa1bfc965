"""Smearing with all steps in one launch against one launch per step, bit for
bit, at the step numbers from which slices of each kind go that way."""
import os

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


@pytest.mark.parametrize("prec", ["F32", "F64"])
@pytest.mark.parametrize("dims,nsteps", [((8, 8, 8, 6), 6), ((10, 6, 10, 4), 6), ((2, 2, 2, 512), 2), ((2, 2, 2, 514), 2),
                                         ((6, 4, 4, 6), 3), ((16, 8, 8, 4), 6)])
def test_smearing_ways(su2, dims, nsteps, prec):
    U = inputs.random_config(dims, 82)
    got = []
    for direct in (False, True):
        lat = su2.Lattice(dims, start=su2.COLD, prec=getattr(su2, prec))
        lat.set_links(U)
        if direct:
            os.environ["SU2_NO_GRAPH"] = "1"
        try:
            lat.ape_smear(0.6, nsteps)
        finally:
            os.environ.pop("SU2_NO_GRAPH", None)
        got.append(lat.get_smeared())
        lat.close()
    assert np.array_equal(got[0], got[1])
