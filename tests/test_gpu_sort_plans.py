"""The bucket sort at the edges of its plans: digit widths (8, 9 and 10 bits,
one to three passes), key counts at which the tiles and the adding up of their
counts change (32,768, 65,536 and 131,072), the ways in which the bucket table
is written (by the sort, by the reorder, by a kernel of its own), and runs of
empty buckets.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

import sph_synth as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


GRIDS = [(1, 1, 1), (16, 16, 1), (257, 1, 1), (8, 8, 8), (513, 1, 1), (32, 32, 1), (41, 25, 1), (64, 64, 16), (256, 16, 16),
         (256, 257, 1), (513, 512, 1), (1024, 64, 17)]
COUNTS = {2: (1, 511, 513), 5: (2047, 2049, 32767, 32768, 32769), 9: (65536, 65537), 12: (131071, 131072, 131073)}


@pytest.mark.parametrize("order", ["random", "sorted", "two clumps"])
@pytest.mark.parametrize("dims", GRIDS, ids=lambda d: "x".join(map(str, d)))
def test_permutation_and_bucket_table(dims, order):
    from paper_2310_03596_amd.sim import Sim
    rng = np.random.default_rng(sum(dims))
    cell = 0.125   # exact: a position's bucket is the same in any arithmetic
    for n in (n for c in COUNTS.values() for n in c):
        wl = S.random_cloud(n, seed=730, h=cell / 2)
        c = np.stack([rng.integers(0, d, size=n) for d in dims], 1)
        if order == "two clumps":   # the first and the last bucket, and one in 1,000 anywhere
            some = rng.random(n) < 1e-3
            c = np.where(some[:, None], c, np.where(rng.random(n)[:, None] < 0.5, 0, np.array(dims) - 1))
        wl.x = (c + rng.integers(1, 8, size=(n, 3)) / 8.0) * cell
        wl.grid = dict(origin=(0.0, 0.0, 0.0), dims=dims, cell=cell)
        key = c[:, 0] + dims[0] * (c[:, 1] + dims[1] * c[:, 2])
        if order == "sorted":
            at = np.argsort(key, kind="stable")
            wl.x, key = wl.x[at], key[at]
        sim = Sim(wl, 1)
        sim.build()
        torch.cuda.synchronize()
        perm = np.argsort(key, kind="stable")
        what = f"{dims} n={n} {order}"
        assert np.array_equal(sim.perm.cpu().numpy(), perm), what
        assert np.array_equal(sim.A.hash.cpu().numpy().view(np.uint32), key[perm]), what
        start = np.searchsorted(key[perm], np.arange(int(np.prod(dims)) + 1))
        assert np.array_equal(sim.start.cpu().numpy(), start), what
        assert np.array_equal(sim.A.id.cpu().numpy(), np.asarray(wl.id)[perm]), what
    print(f"[sort plans] {dims} {order}", flush=True)
