"""APE smearing of small time slices, all steps in one launch, against one
launch per step: bit for bit, and the Wilson loops that follow."""
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
@pytest.mark.parametrize("dims,nsteps", [
    ((2, 2, 2, 2), 3),      # the smallest slice: neighbours on both sides coincide
    ((6, 4, 2, 6), 7),      # 48 sites: one partly filled wavefront
    ((8, 8, 8, 6), 4),      # the largest slice of binary64, 512 sites
    ((10, 6, 10, 4), 2),    # 600 sites: a partly filled wavefront
    ((16, 8, 8, 4), 5),     # the largest slice of binary32, 1024 sites
    ((16, 8, 10, 4), 5),    # beyond it: one launch per step
])
def test_slices_match_steps(su2, dims, nsteps, prec):
    U = inputs.random_config(dims, 81)
    got = []
    for direct in (False, True):
        lat = su2.Lattice(dims, start=su2.COLD, prec=getattr(su2, prec))
        lat.set_links(U)
        if direct:
            os.environ["SU2_NO_GRAPH"] = "1"
        try:
            for k in (nsteps, 1, nsteps + 1):   # the buffers change roles between the calls
                lat.ape_smear(0.6, k)
        finally:
            os.environ.pop("SU2_NO_GRAPH", None)
        got.append((lat.get_smeared(), lat.wilson_loops(2, 2)))
        lat.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
