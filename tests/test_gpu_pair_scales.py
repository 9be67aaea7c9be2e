"""Neighbour sets do not depend on the unit of length: a cloud whose lengths
are all multiplied by a power of two has the same ones, in a run in tiny units
and where (2h)^2 is above 1e30.  Counts and checksums are integers, and a
power of two changes no rounding, so they are equal to those at scale 1 in
both forms."""
import numpy as np
import pytest
import torch

import sph_synth as S

pytestmark = pytest.mark.gpu

PRECS = [pytest.param(0, id="fp64"), pytest.param(1, id="fp32split")]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _census(n, box, scale, prec):
    from paper_2310_03596_amd.sim import Sim
    wl = S.random_cloud(n, seed=760 + n, h=0.0625, box=box)   # buckets of 1/8: exact at every scale
    wl.x = wl.x * scale
    wl.grid = dict(wl.grid, cell=wl.grid["cell"] * scale)
    wl.params = dict(wl.params, h=wl.params["h"] * scale)
    sim = Sim(wl, prec)
    sim.build()
    cnt, chk = sim.census()
    order = np.argsort(sim.A.host()["id"])
    return cnt[order], chk[order]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("exponent", [-40, 57])
@pytest.mark.parametrize("n,box", [(700, 0.5), (5000, 1.0), (40000, 2.0)])   # each width of the pair kernel
def test_power_of_two_units(n, box, exponent, prec):
    ref = _census(n, box, 1.0, prec)
    assert ref[0].min() >= 1   # each finds itself
    print(f"[scales] n={n} 2^{exponent} prec={prec}", flush=True)
    got = _census(n, box, 2.0 ** exponent, prec)
    differ = int(((got[0] != ref[0]) | (got[1] != ref[1])).sum())
    assert differ == 0, f"{differ} of {n} neighbour sets differ"
