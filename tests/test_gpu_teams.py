"""GPU tests of who walks a chunk: one wave to the end, one wave that parks
its walk for a block of eight to go on with, or a block from the start (of
eight waves, or of four where the chunks are many).  The staged records,
tiles and order of summation are the same, so every output has to be bitwise
the same; the split chunks of test_gpu_pieces are switched off, as they add
their sums in another order.

A set of uneven density alone is walked by blocks; next to a set of one level
with small cells it is walked by waves, which park the walks of its dense
clump (several thousand partner records each, every chunk handed out at once).
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

from _checks import check_density, check_force, run_fixed  # noqa: E402

F_KEYS = ("ax", "ay", "az", "dudt", "vsig", "S", "nforce", "hash")


@pytest.fixture(scope="module")
def sph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1309_3783_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def ctx(sph):
    return sph.Context(0)


def _plain():
    return I.fixed_h_case(sphinputs.uniform(500, 93, velocity=True))


def _same(a, b):
    for k in a[0]:
        assert np.array_equal(a[0][k], b[0][k]), k
    for k in F_KEYS:
        assert np.array_equal(a[1][k], b[1][k]), k


# 4500 / 9001: blocks of eight; 75001: 1024 chunks are exceeded, blocks of four
@pytest.mark.parametrize("kind,n", [("mixture", 4500), ("clump", 9001), ("mixture", 75001)])
def test_blocks_equal_waves(sph, ctx, kind, n):
    if kind == "clump":
        ps = sphinputs.clump_by_face(n // 4, n - n // 4, 91, velocity=True)
    else:
        ps = sphinputs.plummer_mixture(n, 97, velocity=True)
    if n <= 10000:
        ps, h = I.fixed_h_case(ps)
    else:
        h = I.f32(ps.h0)
    u, hu = _plain()
    (alone,), _ = run_fixed(sph, ctx, [ps], [h], piece_records=-1)
    both, tree = run_fixed(sph, ctx, [ps, u], [h, hu], piece_records=-1)
    assert tree.stats()["levels"] > 1
    _same(alone, both[0])
    if n <= 10000:
        rd, rf = I.oracle_reference(ps, h)
        check_density(ps, h, alone[0], rd)
        check_force(ps, alone[1], rf)


def test_no_room_to_park(sph, ctx):
    """A workspace without room for the slots of parked walks: the waves walk
    to the end, with the same results."""
    ps, h = I.fixed_h_case(sphinputs.clump_by_face(2000, 7000, 91, velocity=True))
    u, hu = _plain()
    prm = sph.params(flags=sph.SPH_FLAG_PAIR_HASH, piece_records=-1)
    batch = sph.batch_from_sets([ps, u], h=[h, hu])

    def run(nbytes):
        tree = sph.Tree(ctx, workspace=not nbytes)
        if nbytes:
            tree.set_workspace(nbytes)   # (and never grown)
        tree.build_cells(batch, prm)
        tree.sort_pairs()
        dout, fout = sph.DensityOut(batch.n, "cuda", hash=True), sph.ForceOut(batch.n, 2, "cuda", hash=True)
        tree.density(dout)
        tree.force(fout)
        torch.cuda.synchronize()
        r = {k: getattr(dout, k).clone() for k in ("rho", "drho_dh", "nw", "dnw_dh", "nngb", "hash")}
        r.update({k + "_f": getattr(fout, k).clone() for k in F_KEYS})
        return r, tree.workspace_needed(), tree.stats()["chunks"]

    ref, high, chunks = run(0)
    assert 100 < chunks < 2048
    for share in (4, 2):   # of the 4 KiB per chunk that the slots take
        r, used, _ = run(high - 4096 * chunks // share)
        assert used < high
        for k in ref:
            assert torch.equal(ref[k], r[k]), k


def test_density_of_one_level_sets(sph, ctx):
    """A set of one level alone has few chunks, whose density blocks walk; next
    to a larger one waves do."""
    ps, h = I.fixed_h_case(sphinputs.uniform(3001, 94, velocity=True))
    big = sphinputs.uniform(200000, 95)
    (alone,), t1 = run_fixed(sph, ctx, [ps], [h])
    both, t2 = run_fixed(sph, ctx, [big, ps], [I.f32(np.full(big.n, sphinputs.h_for_density(float(big.n)))), h])
    assert t1.stats()["chunks"] < 2048 < t2.stats()["chunks"] and t2.stats()["levels"] == 1
    _same(alone, both[1])
    rd, rf = I.oracle_reference(ps, h)
    check_density(ps, h, alone[0], rd)
    check_force(ps, alone[1], rf)
