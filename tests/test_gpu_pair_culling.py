"""The culling of a window's sources by the box of its targets, before their
records are read: windows none of whose sources are near (of several groups
in turn), windows around one batch of entries (1,536) and two, and boxes
stretched by targets far apart in one bucket row.

The neighbour sets of targets among separate sources are compared exactly
(tests/census.py)."""
import numpy as np
import pytest
import torch

import sph_synth as S
from tests.test_gpu_census import check_census

pytestmark = pytest.mark.gpu

PRECS = [pytest.param(0, id="fp64"), pytest.param(1, id="fp32split")]
H, BOX = 0.05, 1.0   # buckets of 0.1


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _cloud(n, lo, hi, seed):
    wl = S.random_cloud(n, seed=seed, h=H, box=BOX)
    lo, hi = np.broadcast_to(lo, 3), np.broadcast_to(hi, 3)
    wl.x = lo + (hi - lo) * wl.x / BOX
    return wl


def _cases():
    rng = np.random.default_rng(710)
    far = _cloud(60, 0.0, 0.01, 711)                    # 0.14 from the nearest source, in the next bucket
    far.x[20:40] += [0.5, 0.0, 0.0]
    far.x[40:] += [0.0, 0.0, 0.5]
    near = _cloud(300, 0.15, 0.2, 712)
    yield "none near", far, near
    half = _cloud(60, 0.0, 0.01, 711)
    half.x[20:40] += [0.2, 0.2, 0.2]                    # this bucket row has near sources, the first has none
    half.x[40:] += [0.0, 0.5, 0.0]
    yield "one group near", half, near
    for n in (1535, 1536, 1537, 3073):
        yield f"{n} entries", _cloud(70, 0.32, 0.38, 713), _cloud(n, 0.25, 0.45, 714 + n)
    ends = _cloud(64, 0.42, 0.48, 720)
    ends.x[:, 0] = np.where(rng.random(64) < 0.5, 0.03, 0.97)
    yield "far apart in a row", ends, _cloud(9000, 0.0, 1.0, 721)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("case", range(7))
def test_culled_windows(case, prec):
    from paper_2310_03596_amd import _lib as L
    from paper_2310_03596_amd.sim import Sim
    from paper_2310_03596_amd.state import stream_handle
    name, wt, ws = list(_cases())[case]
    t, s = Sim(wt, prec), Sim(ws, prec)
    t.build()
    s.build()
    print(f"[culling] {name} prec={prec} targets={t.n} sources={s.n}", flush=True)
    dev = t.A.x.device
    tidx = torch.arange(t.n, dtype=torch.int32, device=dev)
    nt = torch.tensor([t.n], dtype=torch.int32, device=dev)
    cnt = torch.zeros(t.n, dtype=torch.int32, device=dev)
    chk = torch.zeros(t.n, dtype=torch.int64, device=dev)
    L.sph_neighbor_census(t.params, t.grid, L.SPH_PASS_FORCE, t.A.struct(), tidx.data_ptr(), nt.data_ptr(),
                          s.A.struct(), s.cells, cnt.data_ptr(), chk.data_ptr(), s.ws.data_ptr(), s.ws_bytes,
                          stream_handle())
    torch.cuda.synchronize()
    ht, hs = t.A.host(), s.A.host()
    c, k = cnt.cpu().numpy().view(np.uint32), chk.cpu().numpy().view(np.uint64)
    if name == "none near":
        assert not c.any()
    check_census(c, k, np.arange(t.n), ht["x"], hs["x"], hs["id"], H, prec, name)
