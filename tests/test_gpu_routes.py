"""GPU tests that the routes of the interaction passes are taken at all: which
stages blocks walk from the start, that waves park walks where they may
(sph_tree_stats, sph_last_parked), and that a parked walk ends with bitwise
the results of the wave that has no room to park it.  Besides fixed h: through
the h solve, a solve resumed after a rebuild, a graph, with a halo, with split
chunks, with the pair hashes off, and with several frames in one chunk.

Also the h solve of thousands of sets, whose read-back counts lie next to the
solve's status words.
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

D_KEYS = ("rho", "drho_dh", "nw", "dnw_dh", "nngb", "h", "hash")
F_KEYS = ("ax", "ay", "az", "dudt", "vsig", "S", "nforce", "hash", "sums")


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
    """A set of one level with small cells: next to it waves walk the others."""
    return sphinputs.uniform(500, 93, velocity=True)


def _balls():
    """Eight balls of 6007 particles far apart in one top cell, each within h of
    its own particles alone: a chunk across two balls has a frame in each, with
    about a hundred tiles."""
    rng = np.random.default_rng(5)
    one = sphinputs.clump_by_face(8, 6007, 5, radius=0.01, centre=(0.1, 0.1, 0.1), velocity=True)
    k = np.arange(one.n) >= 8
    cols = {c: np.tile(getattr(one, c)[k], 8) for c in ("m", "u", "vx", "vy", "vz", "h0")}
    at = np.array([[a, b, c] for a in (0.0, 0.25) for b in (0.0, 0.25) for c in (0.0, 0.25)])
    pos = (np.stack([one.x[k], one.y[k], one.z[k]], 1)[None] + at[:, None]).reshape(-1, 3)
    order = rng.permutation(pos.shape[0])
    pos = pos[order]
    ps = sphinputs.ParticleSet(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), cols["m"], cols["u"],
                               *(cols[c][order] for c in ("vx", "vy", "vz")), np.full(pos.shape[0], 0.025), 1.0, {})
    return ps, I.f32(np.full(ps.n, 0.025)), dict(top_grid=2, n_split=1 << 30)


def _pass(sph, ctx, batch, prm, mode, nbytes=None, halo=None, hash=True):
    """One pass of the path; the results, the tree and the walks parked (by the
    last solve or density call, and by the force)."""
    from paper_1309_3783_amd import pipeline as P
    tree = sph.Tree(ctx, workspace=nbytes is None)
    if nbytes is not None:
        tree.set_workspace(nbytes)   # (and never grown)
    out = P.Outputs(batch.n, batch.nsets, hash=hash)
    for k in D_KEYS + F_KEYS:        # (entries of halo particles are not written)
        for o in (out.d, out.f):
            if getattr(o, k, None) is not None:
                getattr(o, k).zero_()
    if mode == "graph":
        P.launch_graph(tree, batch, prm, out, 8)
    else:
        if mode == "solve":
            st, left, _ = sph.solve_with_rebuild(tree, batch, prm, out.d, halo=halo)
            assert st == sph.SPH_OK and left == 0
        else:
            tree.build_cells(batch, prm)
            if halo is not None:
                tree.set_halo(*halo)
            tree.sort_pairs()
            tree.density(out.d)
        tree.force(out.f)
    parked = ctx.parked()
    torch.cuda.synchronize()
    r = {k: getattr(out.d, k).clone() for k in D_KEYS if getattr(out.d, k) is not None}
    r.update({"f_" + k: getattr(out.f, k).clone() for k in F_KEYS if getattr(out.f, k) is not None})
    return r, tree, parked


def _tight(sph, ctx, tree, *args, **kw):
    """The pass in the smallest workspace that it is not refused in, from what
    it needs without the slots on, in steps of 64 KiB."""
    need = tree.workspace_needed() - 4096 * tree.stats()["park_slots"]
    for nbytes in range(need, need + (16 << 20), 65536):
        try:
            return _pass(sph, ctx, *args, nbytes=nbytes, **kw)
        except sph.SphError as e:
            assert e.code == sph.SPH_E_WORKSPACE, e
    raise AssertionError("refused up to 16 MiB beyond the need")


def _same(a, b, n=None):
    for k in a:
        x, y = (a[k], b[k]) if n is None or k == "f_sums" else (a[k][:n], b[k][:n])
        assert torch.equal(x, y), k


CASES = {
    "fixed": dict(n=9001, mode="fixed"),
    "fixed_75k": dict(n=75001, mode="fixed", hash=False),
    "frames": dict(n=0, mode="fixed"),
    "solve": dict(n=30011, mode="solve", prm=dict(h_slack=1.0)),
    "resume": dict(n=30011, mode="solve", prm=dict(h_slack=0.02)),
    "halo": dict(n=30011, mode="solve", prm=dict(h_slack=1.0), halo=True),
    "pieces": dict(n=75001, mode="solve", prm=dict(h_slack=1.0, piece_records=16384)),
    "graph": dict(n=30011, mode="graph", prm=dict(h_slack=1.0)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_parked_walks(sph, ctx, name):
    c = CASES[name]
    hash = c.get("hash", True)
    kw = {"piece_records": -1, **c.get("prm", {})}
    u = _plain()
    if name == "frames":
        ps, h, more = _balls()
        kw.update(more)
    else:
        if name == "pieces":         # (walks of every length: some are split, some parked)
            ps = sphinputs.plummer_mixture(c["n"], 97, velocity=True)
        else:
            ps = sphinputs.clump_by_face(c["n"] // 4, c["n"] - c["n"] // 4, 91, velocity=True)
        h = I.f32(ps.h0)
    prm = sph.params(flags=sph.SPH_FLAG_PAIR_HASH if hash else 0, **kw)
    batch = sph.batch_from_sets([ps, u], h=[h, I.f32(u.h0)])
    halo = None
    if c.get("halo"):
        owned = batch.x < 0.6
        owned[ps.n:] = True
        rho = torch.full_like(batch.h, 1.0)
        halo = (owned.to(torch.uint8), rho, -3.0 * rho / batch.h)
    args = (batch, prm, c["mode"])
    ref, tree, parked = _pass(sph, ctx, *args, halo=halo, hash=hash)
    st = tree.stats()
    print(name, "chunks", st["chunks"], "slots", st["park_slots"], "parked", parked, "builds", tree.builds)
    assert st["block_walks"] == 0 and st["park_slots"] == min(st["chunks"], 2048)
    assert parked[0] > 0 and parked[1] > 0
    assert (tree.builds > 1) == (name == "resume")
    assert (st["pieces"] > 0) == (name == "pieces")
    got, tight, none = _tight(sph, ctx, tree, *args, halo=halo, hash=hash)
    assert tight.stats()["park_slots"] == 0 and none == (0, 0)
    _same(got, ref)
    if name in ("pieces", "halo"):
        return
    # the set alone: blocks walk its chunks, in the same order of summation
    alone = sph.batch_from_sets([ps], h=[h])
    got, tree, parked = _pass(sph, ctx, alone, prm, c["mode"], hash=hash)
    st = tree.stats()
    assert st["block_walks"] == 3 and st["park_slots"] == 0 and parked == (0, 0)
    got.pop("f_sums")
    ref.pop("f_sums")
    _same(got, ref, ps.n)


def test_blocks_walk_the_density_of_small_sets(sph, ctx):
    u = sphinputs.uniform(3001, 94)
    _, tree, parked = _pass(sph, ctx, sph.batch_from_sets([u]), sph.params(), "fixed", hash=False)
    assert tree.stats()["block_walks"] == 1 and tree.stats()["park_slots"] == 0 and parked == (0, 0)
    u = sphinputs.uniform(200000, 95)
    _, tree, parked = _pass(sph, ctx, sph.batch_from_sets([u]), sph.params(), "fixed", hash=False)
    assert tree.stats()["block_walks"] == 0 and tree.stats()["park_slots"] == 0 and parked == (0, 0)


@pytest.mark.parametrize("nsets", [2800, 4096])
def test_solve_of_many_sets(sph, nsets):
    """The extremes of h of more than 2730 sets take more than 32 KiB of the
    pinned memory (12 bytes a set; 4096 sets are the most): the solves before
    and after a build wait for their own words, and each set ends as it would
    with seven others."""
    few = [sphinputs.uniform(300 + k % 3, 700 + k) for k in range(8)]
    prm = sph.params(h_slack=1.0)
    ctx = sph.Context(0)

    def solve(tree, sets):
        batch = sph.batch_from_sets(sets)
        got = []
        for _ in range(2):
            tree.build_cells(batch, prm)
            tree.sort_pairs()
            d = sph.DensityOut(batch.n, "cuda")
            st, left, it = tree.solve_h(d)
            assert st == sph.SPH_OK and left == 0
            got.append((d.h.clone(), d.nngb.clone(), it))
        assert torch.equal(got[0][0], got[1][0]) and got[0][2] == got[1][2]
        return got[0]

    h1, n1, it1 = solve(sph.Tree(ctx), few)
    h2, n2, it2 = solve(sph.Tree(ctx), few * (nsets // 8))
    assert torch.equal(h1.repeat(nsets // 8), h2) and torch.equal(n1.repeat(nsets // 8), n2) and it1 == it2
