"""The pair kernel's widths (4, 8 and 16 targets per wavefront, by the size of
the call): neighbour sets around the changes, in windows longer than a batch
with more hits per target than one round lists, exactly; and each pass over
copies of a body far apart, which must give every particle of the first copy
what the body alone gives, up to the order of the FP64 summation."""
import numpy as np
import pytest
import torch

import sph_synth as S
from tests.test_gpu_census import check_census

pytestmark = pytest.mark.gpu

PRECS = [pytest.param(0, id="fp64"), pytest.param(1, id="fp32split")]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n", [12288, 12289, 16385, 24577, 32769])
def test_neighbour_sets_of_each_width(n, prec):
    from paper_2310_03596_amd.sim import Sim
    wl = S.random_cloud(n, seed=740, h=0.05, box=0.6)   # 57 to 152 particles a bucket, 240 to 640 neighbours
    print(f"[tiles] n={n} prec={prec}", flush=True)
    sim = Sim(wl, prec)
    sim.build()
    cnt, chk = sim.census()
    h = sim.A.host()
    t = np.unique(np.concatenate([np.arange(200), np.arange(n - 200, n), np.random.default_rng(741).integers(0, n, 600)]))
    check_census(cnt, chk, t, h["x"][t], h["x"], h["id"], wl.params["h"], prec, f"n={n}")


def _copies(wl, k):
    """k copies of wl, 8 buckets of empty space apart along x, on the grid of 9."""
    L = wl.grid["cell"]
    width = wl.grid["dims"][0] + 8
    out = S.Workload(wl.name, *[np.concatenate([f] * k) for f in (wl.x, wl.v, wl.m, wl.omega, wl.rho, wl.E)],
                     np.arange(k * wl.n, dtype=wl.id.dtype), dict(wl.grid, dims=(9 * width, *wl.grid["dims"][1:])),
                     wl.params, extra=wl.extra)
    for c in range(1, k):
        out.x[c * wl.n:(c + 1) * wl.n, 0] += c * width * L
    if wl.S is not None:
        out.S, out.eps_p = np.concatenate([wl.S] * k), np.concatenate([wl.eps_p] * k)
    return out


def _passes(wl, n, prec, solid):
    """Outputs of every pass for the particles with id < n, in id order."""
    from paper_2310_03596_amd import _lib as L
    from paper_2310_03596_amd.adjoint import Cotangent
    from paper_2310_03596_amd.sim import Sim
    from paper_2310_03596_amd.state import Rates, stream_handle
    sim = Sim(wl, prec)
    sim.build()
    ids = sim.A.id.long()
    pick = torch.argsort(ids)[:n]
    out = {}
    for pass_ in (0, 1) if solid else (0,):
        sim.interact(pass_=pass_)
        out[f"pass {pass_}"] = (sim.rates.grad() if pass_ else sim.rates.force())[:, pick].cpu().numpy()
        rbar, bar = Rates(sim.n, prec, solid, "cuda"), Cotangent(sim.n, prec, "cuda", solid)
        rng = np.random.default_rng(742)
        for name in ("hi", "Lhi"):
            t = getattr(rbar, name)
            if t is not None:
                by_id = torch.from_numpy(rng.normal(size=(t.shape[0], n))).to(t)
                t.copy_(by_id[:, ids % n])
        a, r = sim.A.struct(), rbar.struct()
        wsb = L.sph_workspace_size(sim.grid, sim.n, prec, L.SPH_SOLID_J2)
        ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
        L.sph_interact_adjoint(sim.params, sim.grid, pass_, a, None, None, a, sim.cells, r, r, bar.struct(),
                               ws.data_ptr(), wsb, stream_handle())
        torch.cuda.synchronize()
        for f in ("x", "v", "w") + (() if pass_ else ("rho", "p", "c", "e")) + (("S",) if solid and not pass_ else ()):
            out[f"reverse {pass_} {f}"] = getattr(bar, f).double().reshape(-1, sim.n)[:, pick].cpu().numpy()
    return out


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("solid", [False, True], ids=["fluid", "solid"])
def test_copies_agree(solid, prec):
    wl = S.solid_block(16, seed=743, s_sigma=1e7) if solid else S.jittered_lattice(16, seed=744, jitter=0.2)
    assert wl.n == 4096
    ref = _passes(_copies(wl, 1), wl.n, prec, solid)
    for k in (2, 3, 5, 9):
        got = _passes(_copies(wl, k), wl.n, prec, solid)
        print(f"[copies] {k} x {wl.n} solid={solid} prec={prec}", flush=True)
        for f, want in ref.items():
            # the terms are the same: about 80 FP64 additions of terms that may
            # cancel, by a factor that stays far below 1e3, to a result of the
            # field's size; a reverse pass stores in the form's precision
            tol = 80 * 2.0 ** -53 * 1e3 * np.abs(want).max(axis=1, keepdims=True)
            if prec == 1:
                tol = tol + 2.0 ** -23 * np.abs(want)
            assert (np.abs(got[f] - want) <= tol).all(), (k, f, np.abs(got[f] - want).max(), np.abs(want).max())
