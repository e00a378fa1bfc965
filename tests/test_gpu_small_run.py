"""Whole runs of small lattices in one launch (one workgroup per lattice, links
in LDS) against the same sweeps launched substep by substep: links, try counts
and sweep counter bit for bit, series up to the rounding of their sums (1e-14:
sums of at most 6144 terms of order 1, compensated or by wavefront)."""
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


class Direct:
    def __enter__(self):
        os.environ["SU2_NO_GRAPH"] = "1"

    def __exit__(self, *a):
        os.environ.pop("SU2_NO_GRAPH", None)


SHAPES = [
    [(2, 2, 2, 2)],                              # 8 links a substep
    [(4, 4, 4, 4)],
    [(8, 4, 4, 8)],                              # the largest of binary32: 1024 sites
    [(8, 4, 4, 4)],                              # the largest of binary64: 512 sites
    [(2, 6, 10, 4)],                             # 240 links: a partial wavefront
    [(4, 4, 4, 6), (2, 2, 2, 2), (6, 4, 4, 10)],  # uneven, one launch
    [(4, 4, 4, 4)] * 300,                        # two workgroups on a compute unit
]


@pytest.mark.parametrize("prec", ["F32", "F64"])
@pytest.mark.parametrize("dims", SHAPES, ids=lambda d: "%dx%s" % (len(d), "x".join(map(str, d[0]))))
def test_small_runs_match_substeps(su2, dims, prec):
    betas = [2.0 + 0.5 * i / len(dims) for i in range(len(dims))]
    got = []
    for direct in (False, True):
        ens = su2.Ensemble(dims, betas, start=su2.HOT, seed=21, prec=getattr(su2, prec))
        if direct:
            with Direct():
                series = [ens.run(n, seed, measure_every=e) for n, e, seed in ((7, 1, 21), (1, 1, 21), (11, 3, 22))]
        else:
            series = [ens.run(n, seed, measure_every=e) for n, e, seed in ((7, 1, 21), (1, 1, 21), (11, 3, 22))]
        # a run that records its tries goes substep by substep on the same counter
        ens.trace_tries(True)
        ens.run(2, 22)
        got.append((series, [ens.get_links(i) for i in range(len(dims))], ens.stats(), ens.get_tries(0)))
        ens.close()
    a, b = got
    for (p, q), (p2, q2) in zip(a[0], b[0]):
        assert np.abs(p - p2).max() < 1e-14 and np.abs(q - q2).max() < 1e-14
    assert all(np.array_equal(x, y) for x, y in zip(a[1], b[1]))
    assert a[2] == b[2] and np.array_equal(a[3], b[3])


@pytest.mark.parametrize("prec", ["F32", "F64"])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 6, 6, 2), (4, 4, 4, 4), (4, 4, 4, 6), (8, 4, 4, 8)])
def test_small_updates_match_substeps(su2, dims, prec):
    """Heat bath (both samplers) mixed with over-relaxation on a lattice of
    given links."""
    U = inputs.random_config(dims, 71)
    got = []
    for direct in (False, True):
        lat = su2.Lattice(dims, start=su2.COLD, prec=getattr(su2, prec))
        lat.set_links(U)
        for sampler in (su2.HYBRID, su2.CREUTZ):
            su2.su2_set_sampler(lat.h, sampler)
            if direct:
                with Direct():
                    lat.heatbath(2.3, 2, 5)
                    lat.overrelax(3)
            else:
                lat.heatbath(2.3, 2, 5)
                lat.overrelax(3)
        got.append((lat.get_links(), lat.sweep, lat.stats()[:2], lat.plaquette(), lat.polyakov()))
        lat.close()
    a, b = got
    assert np.array_equal(a[0], b[0]) and a[1:] == b[1:]


def test_small_run_reports_nonfinite(su2):
    """A non-finite link is counted by the run that meets it, and reported
    once, also by over-relaxation."""
    import torch
    for over in (False, True):
        lat = su2.Lattice((4, 4, 4, 4), start=su2.HOT, seed=3, prec=su2.F32)
        # a temporal link: a sweep redraws the x links first, from staples that hold it
        lat._buf.view(torch.float32).view(8, -1)[6, :4] = float("nan")
        torch.cuda.synchronize()
        with pytest.raises(su2.SU2Error) as e:
            lat.overrelax(1) if over else lat.heatbath(2.3, 1, 3)
        assert e.value.status == su2.ENUMERIC
        lat.polyakov()   # the count was cleared
        lat.close()
