"""GPU tests at the sizes where the build and the h solve change their kernels.

* The particles' sort: all passes in one block up to 12288, blocks that add up
  the histograms themselves up to 64 blocks of 4096, a scanned histogram
  beyond; a wrong order loses partners (pair hashes against the oracle).
* The Newton step and the counts of particles still active: one kernel up to
  64 reduction chunks (a set has at least one), separate kernels beyond; a
  set's h and the counts have to be the same.
"""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
import _inputs as I  # noqa: E402

import sphinputs  # noqa: E402

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from _checks import check_density, run_fixed  # noqa: E402


@pytest.fixture(scope="module")
def sph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1309_3783_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("n", [2, 1024, 1025, 12288, 12289, 262144, 262145])
def test_sort_of_particles(sph, n):
    ps = sphinputs.uniform(n, 21)
    h = I.f32(np.full(n, min(0.3, sphinputs.h_for_density(float(n)))))
    if n > 1000:
        ps = I.redraw_ties_uniform(ps, h, seed=22)
    (res,), _ = run_fixed(sph, sph.Context(0), [ps], [h])
    import oracle
    rd = oracle.density(ps.x, ps.y, ps.z, h, ps.m, ps.box)
    check_density(ps, h, res[0], rd)


@pytest.mark.parametrize("max_iter", [3, 30])
def test_newton_counts(sph, max_iter):
    sets = [sphinputs.uniform(600 + k, 500 + k) for k in range(65)]
    prm = sph.params(max_iter=max_iter, h_slack=1.0)

    def solve(which):
        batch = sph.batch_from_sets([sets[k] for k in which])
        tree = sph.Tree(sph.Context(0))
        tree.build_cells(batch, prm)
        tree.sort_pairs()
        out = sph.DensityOut(batch.n, "cuda")
        _, left, _ = tree.solve_h(out)
        torch.cuda.synchronize()
        return out.h.cpu().numpy(), left

    h65, left65 = solve(range(65))     # 65 chunks: separate kernels
    h64, left64 = solve(range(64))     # 64 chunks: one kernel
    h1, left1 = solve([64])
    assert np.array_equal(h65, np.concatenate([h64, h1]))
    assert left65 == left64 + left1
    assert (left65 > 0) == (max_iter == 3)



def test_counts_of_many_sets(sph):
    """The h extremes of 3000 sets are read back in one piece (36 KB)."""
    few = [sphinputs.uniform(120 + k % 3, 700 + k) for k in range(6)]
    prm = sph.params(h_slack=1.0, max_iter=3)

    def solve(sets):
        batch = sph.batch_from_sets(sets)
        tree = sph.Tree(sph.Context(0))
        for _ in range(2):
            tree.build_cells(batch, prm, h=None)
            tree.sort_pairs()
            out = sph.DensityOut(batch.n, "cuda")
            tree.density(out)
        torch.cuda.synchronize()
        return out.rho.cpu().numpy(), out.nngb.cpu().numpy()

    r1, n1 = solve(few)
    r2, n2 = solve(few * 500)
    assert np.array_equal(np.tile(r1, 500), r2) and np.array_equal(np.tile(n1, 500), n2)
