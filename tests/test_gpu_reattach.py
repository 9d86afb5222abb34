"""GPU tests of a tree whose memory is replaced: another workspace attached,
library-owned buffers exchanged for a workspace, the static scratch taken back
from another tree.  Nothing may work through pointers into the memory before:
the old workspace keeps a pattern written to it, and the results are bitwise
those of a fresh tree.
"""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(__file__))

import sphinputs  # noqa: E402

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1309_3783_amd as m
    m.lib()
    return m


def _batch(sph, n, seed):
    return sph.batch_from_sets([sphinputs.plummer_mixture(n, seed, velocity=True, snap=False)])


def _run(sph, tree, batch, prm, build=None):
    from paper_1309_3783_amd import pipeline as P
    out = P.Outputs(batch.n, batch.nsets, hash=True)
    (build or tree.build_cells)(batch, prm)
    tree.sort_pairs()
    st, _, _ = tree.solve_h(out.d)
    assert st == sph.SPH_OK
    tree.force(out.f)
    torch.cuda.synchronize()
    r = {k: getattr(out.d, k).clone() for k in ("rho", "drho_dh", "nw", "dnw_dh", "nngb", "h", "hash")}
    r.update({"f_" + k: getattr(out.f, k).clone() for k in ("ax", "ay", "az", "dudt", "vsig", "S", "nforce", "hash")})
    return r


def _same(a, b):
    for k in a:
        assert torch.equal(a[k], b[k]), k


# the second batch smaller, and somewhat larger (within the scratch of the first's sort)
@pytest.mark.parametrize("n2", [9000, 33000])
@pytest.mark.parametrize("owned_first", [False, True])
def test_another_workspace(sph, n2, owned_first):
    ctx = sph.Context(0)
    prm = sph.params(flags=sph.SPH_FLAG_PAIR_HASH, h_slack=0.5)
    one, two = _batch(sph, 30000, 41), _batch(sph, n2, 42)
    size = sph.workspace_size(33000, 1, prm)
    tree = sph.Tree(ctx, workspace=False)
    if not owned_first:
        tree.set_workspace(size)
        first = tree.ws
    _run(sph, tree, one, prm)
    tree.set_workspace(size)
    if not owned_first:
        torch.cuda.synchronize()
        first.fill_(0xA5)
    got = _run(sph, tree, two, prm)
    _same(got, _run(sph, sph.Tree(ctx), two, prm))
    if not owned_first:
        assert bool((first == 0xA5).all())


def test_static_scratch_taken_back(sph):
    ctx = sph.Context(0)
    prm = sph.params(flags=sph.SPH_FLAG_PAIR_HASH, h_slack=0.5)
    one, two = _batch(sph, 20000, 43), _batch(sph, 15000, 44)
    a, b = sph.Tree(ctx, workspace=False), sph.Tree(ctx, workspace=False)
    _run(sph, a, one, prm, a.build_cells_static)
    _run(sph, b, one, prm, b.build_cells_static)
    got = _run(sph, a, two, prm, a.build_cells_static)
    _same(got, _run(sph, sph.Tree(ctx), two, prm))
