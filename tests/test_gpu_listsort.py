"""GPU test of the sorts of the cells' particle lists at the sizes where the
sort changes: 64 K entries fill a wave's K registers per lane (K = 2, 4, 8), a
block merges runs up to 1024, 2048 and 4096 entries, a large block up to 8192
and 16384.  Two top cells per side hold an exact number of particles each;
every list is sorted (no partner is read in cell order), and a wrong order
loses partners of the sweeps, which the pair hashes show.
"""
import dataclasses
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


@pytest.mark.parametrize("counts", [(64, 65, 128, 129, 256, 257, 512, 513),
                                    (1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193)])
def test_lists_at_the_sorts_edges(sph, counts):
    ps = sphinputs.uniform(sum(counts), 17, velocity=True)
    at = np.repeat(np.arange(8), counts)
    half = 0.5 * ps.box
    ps = dataclasses.replace(ps, x=0.5 * ps.x + half * (at & 1), y=0.5 * ps.y + half * (at >> 1 & 1),
                             z=0.5 * ps.z + half * (at >> 2))
    # two sizes of h: both parts of the lists have entries
    h = np.where(np.arange(ps.n) % 7 == 0, 0.11, 0.05) * ps.box
    ps, h = I.fixed_h_case(ps, I.f32(h))
    (res,), tree = run_fixed(sph, sph.Context(0), [ps], [h], flags=sph.SPH_FLAG_SORTED_ONLY, top_grid=2,
                             n_split=1 << 30)
    st = tree.stats()
    assert st["top_grid"] == 2 and st["levels"] == 1 and st["max_leaf"] == max(counts), st
    rd, rf = I.oracle_reference(ps, h)
    check_density(ps, h, res[0], rd)
    # (the force values are no measure here: particles with one partner have a
    # grad-h factor near zero, which no FP32 density resolves)
    assert np.array_equal(res[1]["nforce"], rf["nforce"])
    assert np.array_equal(res[1]["hash"], rf["hash"])
