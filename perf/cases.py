"""Timed cases of the SPH density/force path, through the package's own entry points.

A case is one particle workload and the way a program drives it:

* ``fixed``  -- cells, sorted lists, density and force at given smoothing lengths (a caller that keeps h);
* ``solve``  -- cells, sorted lists, the Newton solve of h from a first guess, force (one step of a run);
* ``graph``  -- many independent sets, or one request, in one build and one HIP graph (batched and served);
* ``step``   -- one kick-drift-kick step with its Courant minimum, tree made anew or kept from step to step;
* ``share``  -- one GPU's part of a decomposed set: owned particles plus a read-only halo.

Inputs are drawn on the GPU from the seed: jittered lattices, uniform sets, mixtures of 64 Plummer clumps with a
20% uniform background (h over up to three decades) and the two-density shock tube; periodic unit cubes, equal
masses, positions on the 2^-24 grid, all distinct.  In caller order, as a program holds them."""
import math

import numpy as np
import torch

import paper_1309_3783_amd as sph
from paper_1309_3783_amd import integrate, pipeline

N_NGB, GAMMA, ALPHA = 48.0, 5.0 / 3.0, 2.0
GRID = 1 << 24
K_ITER = 24          # Newton passes captured in a graph, as the batched and served modes use
DENSITY = ("rho", "drho_dh", "nw", "dnw_dh", "nngb", "h", "hash")
FORCE = ("ax", "ay", "az", "dudt", "vsig", "S", "nforce", "hash", "sums")


def listed():
    return [
        # the smallest set of the tests, constant h: launches and read-backs are all it costs
        _case("fixed_uniform_4k", "fixed", "uniform", 4096, velocity=False),
        # a clumpy set with everything asked for: velocities and the pair-set hashes of both stages
        _case("fixed_mixture_30k_hash", "fixed", "mixture", 30011, hash=True),
        # a quarter-million lattice with velocities, an odd number per side
        _case("fixed_lattice_250k", "fixed", "lattice", 63 ** 3),
        # one multi-resolution set of a million at the h of the step before
        _case("fixed_mixture_1m", "fixed", "mixture", 1000003),
        # the smallest request a server is sent: h solved from the first guess
        _case("solve_mixture_10k", "solve", "mixture", 10000, velocity=False),
        # a middle-sized clumpy request
        _case("solve_mixture_200k", "solve", "mixture", 200000, velocity=False),
        # the headline workload: 100^3 lattice jittered by a tenth of the spacing
        _case("solve_lattice_1m", "solve", "lattice", 100 ** 3, velocity=False),
        # the largest: the stand-in for a cosmological volume
        _case("solve_mixture_8m", "solve", "mixture", 8000000, velocity=False),
        # uneven independent sets in one build and one graph
        _case("graph_64_sets", "graph", "mixture", 12000, velocity=False, sets=64),
        # the shock tube of the validation runs, cells made anew each step, Courant minimum read each step
        _case("step_tube_163k", "step", "tube", 163072, velocity=False, dt=2e-5),
        # a moving lattice whose cells and sorted lists are kept from step to step
        _case("step_lattice_1m_reuse", "step", "lattice", 100 ** 3, dt=2e-5, reuse=True),
        # one GPU's part of a decomposed lattice: an eighth of the box and the halo around it
        _case("share_lattice_1m", "share", "lattice", 176 ** 3, velocity=False),
    ]


def _case(name, mode, recipe, n, velocity=True, hash=False, sets=1, dt=0.0, reuse=False):
    c = {"mode": mode, "recipe": recipe, "n": n, "velocity": velocity, "hash": hash, "sets": sets, "dt": dt,
         "reuse": reuse}
    return {"name": name, **c} if name else c


def draw(rng):
    mode = rng.choice(["fixed", "fixed", "solve", "solve", "graph", "step", "share"])
    recipe = rng.choice(["lattice", "mixture", "mixture", "uniform"])

    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | rng.randrange(2)

    velocity = rng.random() < 0.5
    if mode == "graph":
        sets = rng.choice([1, 1, 3, 7, 16, 41, 64, 100])
        c = _case(None, mode, "mixture", size(4000, 800000 if sets == 1 else 30000), velocity, sets=sets)
    elif mode == "step":
        recipe = rng.choice(["tube", "lattice", "mixture"])
        c = _case(None, mode, recipe, size(30000, 1000000), velocity, dt=2e-6 if recipe == "mixture" else 2e-5,
                  reuse=rng.random() < 0.5)
    elif mode == "share":
        c = _case(None, mode, "lattice", size(64 ** 3, 190 ** 3), velocity)
    else:
        c = _case(None, mode, recipe, size(3000, 4000000 if mode == "solve" else 1500000), velocity,
                  hash=rng.random() < 0.25)
    return c


# ---- inputs -------------------------------------------------------------------------------------------------------

def _h_for(density):
    return (3.0 * N_NGB / (4.0 * math.pi) / density) ** (1.0 / 3.0)


def _distinct(pos):
    """Positions as FP64 multiples of 2^-24 in [0, 1), duplicates moved to a free neighbouring point."""
    k = torch.remainder(torch.floor(torch.remainder(pos, 1.0) * GRID).to(torch.int64), GRID)
    while True:
        # an injective key would take 72 bits: a mixed 64-bit one, equal keys taken for equal points
        key = (k[:, 0] * 0x1E3779B97F4A7C15 + k[:, 1]) * 0x3F58476D1CE4E5B9 + k[:, 2]
        s, order = torch.sort(key, stable=True)
        dup = order[1:][s[1:] == s[:-1]]
        if dup.numel() == 0:
            return k.to(torch.float64) / GRID
        k[dup, 2] = torch.remainder(k[dup, 2] + 1, GRID)


def _lattice(n, jitter, g):
    side = max(4, round(n ** (1.0 / 3.0)))
    a = (torch.arange(side, device="cuda", dtype=torch.float64) + 0.5) / side
    pos = torch.stack(torch.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)
    pos = pos + (torch.rand(pos.shape, generator=g, device="cuda", dtype=torch.float64) * 2 - 1) * (jitter / side)
    return pos, torch.full((pos.shape[0],), _h_for(float(pos.shape[0])), device="cuda", dtype=torch.float64)


def _tube(n, g):
    """Two lattices of equal-mass particles, density 1 in x < 1/2 and about 1/4 beyond (64, 40 per side at 163k)."""
    nl = 2 * max(2, round((n / 0.6221) ** (1.0 / 3.0) / 2))
    nr = max(4, round(nl * 40 / 64))
    parts, hs = [], []
    for lo, nx, ny in ((0.0, nl // 2, nl), (0.5, nr // 2, nr)):
        ax = lo + (torch.arange(nx, device="cuda", dtype=torch.float64) + 0.5) * (0.5 / nx)
        ay = (torch.arange(ny, device="cuda", dtype=torch.float64) + 0.5) / ny
        p = torch.stack(torch.meshgrid(ax, ay, ay, indexing="ij"), -1).reshape(-1, 3)
        p = p + (torch.rand(p.shape, generator=g, device="cuda", dtype=torch.float64) * 2 - 1) * (0.02 / ny)
        parts.append(p)
        hs.append(torch.full((p.shape[0],), _h_for(p.shape[0] / 0.5), device="cuda", dtype=torch.float64))
    return torch.cat(parts), torch.cat(hs), parts[0].shape[0]


def _mixture(n, g, clumps=64, background=0.2):
    dev = dict(device="cuda", dtype=torch.float64)
    n_bg = round(background * n)
    per = (n - n_bg) // clumps
    n_bg = n - per * clumps
    a = 10.0 ** (torch.rand(clumps, generator=g, **dev) * 2 - 3)
    rmax = torch.clamp(20 * a, max=0.45)
    umax = rmax ** 3 / (rmax ** 2 + a ** 2) ** 1.5
    centre = torch.rand((clumps, 3), generator=g, **dev)
    u = torch.clamp(torch.rand((clumps, per), generator=g, **dev) * umax[:, None], min=1e-300)
    r = a[:, None] / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
    d = torch.randn((clumps, per, 3), generator=g, **dev)
    d = d / d.norm(dim=-1, keepdim=True)
    pos = torch.cat([torch.rand((n_bg, 3), generator=g, **dev), (centre[:, None] + r[..., None] * d).reshape(-1, 3)])
    pos = torch.remainder(pos, 1.0)
    dens = torch.full((n,), float(n_bg), **dev)
    for c in range(clumps):      # the analytic number density gives the first guess of h
        q = pos - centre[c]
        q -= torch.round(q)
        r2 = (q * q).sum(-1)
        rho = 3.0 * per / (4.0 * math.pi * a[c] ** 3 * umax[c]) * (1.0 + r2 / a[c] ** 2) ** -2.5
        dens += torch.where(r2 < rmax[c] ** 2, rho, 0.0)
    return pos, _h_for(dens)


def _set_sizes(case):
    """One set, or sizes log-uniform over a factor of ten around case["n"]."""
    if case["sets"] == 1:
        return [case["n"]]
    r = np.random.default_rng(case["n"] + case["sets"])
    return [int(v) for v in case["n"] * np.exp(r.uniform(-1.15, 1.15, case["sets"]))]


def _particles(case, seed):
    """Caller-order FP64 positions, FP32 h, m, u, v and the set offsets."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cols, off, box_m = [], [0], []
    for n in _set_sizes(case):
        split = None
        if case["recipe"] == "lattice":
            pos, h = _lattice(n, 0.1, g)
        elif case["recipe"] == "tube":
            pos, h, split = _tube(n, g)
        elif case["recipe"] == "mixture":
            pos, h = _mixture(n, g)
        else:
            pos = torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float64)
            h = torch.full((n,), _h_for(float(n)), device="cuda", dtype=torch.float64)
        pos = _distinct(pos)
        k = pos.shape[0]
        v = (torch.rand((k, 3), generator=g, device="cuda") * 2 - 1) * (0.1 if case["velocity"] else 0.0)
        u = torch.full((k,), 1.5, device="cuda")
        m = torch.full((k,), 1.0 / k, device="cuda")
        if split is not None:    # pressures 1 and 0.1795
            m.fill_(0.5 / split)
            u[split:] = 0.1795 / ((GAMMA - 1.0) * ((k - split) / split))
        cols.append((pos, h.float(), m, u, v))
        off.append(off[-1] + k)
    pos, h, m, u, v = (torch.cat(t) for t in zip(*cols))
    return pos, h, m, u, v, np.array(off, dtype=np.int64)


def _share_of(pos, h):
    """Indices of an eighth of the box and the layer of halo particles around it, and the owned mask (by the
    particles' lattice sites)."""
    side = round(pos.shape[0] ** (1.0 / 3.0))
    site = (torch.floor(pos * side) + 0.5) / side
    layer = 1.0 / 2 ** int(math.log2(1.0 / (1.25 * float(h.max()))))
    near = (torch.remainder(site + layer, 1.0) < 0.5 + 2 * layer).all(-1).nonzero().squeeze(-1)
    return near, (site[near] < 0.5).all(-1)


# ---- a user's program ---------------------------------------------------------------------------------------------

def prepare(case, seed):
    pos, h, m, u, v, off = _particles(case, seed)
    owned = None
    if case["mode"] == "share":
        near, owned = _share_of(pos, h)
        pos, h, m, u, v = pos[near], h[near], m[near], u[near], v[near]
        off = np.array([0, pos.shape[0]], dtype=np.int64)
    x, y, z = (pos[:, k].contiguous() for k in range(3))
    vx, vy, vz = (v[:, k].contiguous() for k in range(3))
    batch = sph.Batch(x, y, z, h, m, u, vx, vy, vz, off, np.ones(len(off) - 1))
    ctx = sph.Context(0)
    prm = sph.params(flags=sph.SPH_FLAG_PAIR_HASH if case["hash"] else 0)
    st = {"mode": case["mode"], "dt": case["dt"], "ctx": ctx, "batch": batch, "prm": prm}
    if case["mode"] == "step":
        st["run"] = integrate.Leapfrog(ctx, batch, prm, reuse=case["reuse"])
        return st
    st["tree"] = sph.Tree(ctx)
    st["out"] = pipeline.Outputs(batch.n, batch.nsets, hash=case["hash"])
    if owned is not None:
        # the halo particles' density as their owners hold it: the lattice's mean
        rho = torch.full_like(h, float(m[0]) * round(1.0 / float(m[0])))
        st["halo"] = (owned.to(torch.uint8), rho, -3.0 * rho / h)
        for t in [getattr(st["out"].d, k) for k in DENSITY] + [getattr(st["out"].f, k) for k in FORCE]:
            if t is not None:
                t.zero_()        # (the entries of halo particles are not written)
    return st


def run(st):
    mode, batch, prm = st["mode"], st["batch"], st["prm"]
    if mode == "step":
        lf = st["run"]
        lf.step(min(st["dt"], lf.cfl_dt()))
        return {"x": batch.x, "y": batch.y, "z": batch.z, "vx": batch.vx, "vy": batch.vy, "vz": batch.vz,
                "u": batch.u, **_returned(lf.d, lf.f)}
    tree, out = st["tree"], st["out"]
    if mode == "graph":
        pipeline.run_graph(tree, batch, prm, out, K_ITER)
        return {"status": out.status, **_returned(out.d, out.f)}
    if mode == "fixed":
        tree.build_cells(batch, prm)
        tree.sort_pairs()
        tree.density(out.d)
    else:
        status, left, _ = sph.solve_with_rebuild(tree, batch, prm, out.d, halo=st.get("halo"))
        if status not in (sph.SPH_OK, sph.SPH_E_NOCONV):
            raise RuntimeError("solve: status %d, %d left" % (status, left))
    tree.force(out.f)
    return _returned(out.d, out.f)


def _returned(d, f):
    got = {k: getattr(d, k) for k in DENSITY if getattr(d, k) is not None}
    got.update({"f_" + k: getattr(f, k) for k in FORCE if getattr(f, k) is not None})
    return got


def _count(case):
    n = case["n"]
    if case["mode"] == "share":
        n = int(n * (0.5 + 4.0 * _h_for(float(n))) ** 3)
    return n * case["sets"]


def work(case):
    """Inputs read once (48 B a particle), outputs written once; per unordered pair one density evaluation of 70
    lane operations and one force evaluation of 125, 24 pairs a particle at 48 neighbours."""
    n = _count(case)
    out = 28 + 28 + (16 if case["hash"] else 0) + (40 if case["mode"] == "step" else 0)
    return {"bytes": n * (48 + out), "flops": n * 24 * 195}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------

def _pairs(pos, h, most=30_000_000):
    """Ordered pairs (i, j), j != i, with r < h_i in the periodic unit cube, in parts: cells of at least h_i."""
    level = torch.floor(-torch.log2(h)).to(torch.int64)
    for lv in torch.unique(level).tolist():
        tgt = (level == lv).nonzero().squeeze(-1)
        lv = lv if lv >= 2 else 0              # fewer than four cells a side: one cell
        G = 1 << lv
        c = torch.clamp((pos * G).to(torch.int64), max=G - 1)
        ids, order = torch.sort((c[:, 0] * G + c[:, 1]) * G + c[:, 2])
        steps = (-1, 0, 1) if lv else (0,)
        off = torch.tensor([(a, b, d) for a in steps for b in steps for d in steps], device=pos.device)
        at = 0
        while at < tgt.numel():
            t = tgt[at:at + max(1, min(tgt.numel(), most // (27 * 8)))]
            nb = torch.remainder(c[t][:, None] + off, G)
            nid = (nb[..., 0] * G + nb[..., 1]) * G + nb[..., 2]
            lo, hi = torch.searchsorted(ids, nid), torch.searchsorted(ids, nid, right=True)
            per = torch.cumsum((hi - lo).sum(-1), 0)
            k = max(1, int(torch.searchsorted(per, most)))
            t, lo, cnt = t[:k], lo[:k].reshape(-1), (hi - lo)[:k].reshape(-1)
            at += k
            i = t.repeat_interleave(off.shape[0]).repeat_interleave(cnt)
            first = torch.cumsum(cnt, 0) - cnt
            j = order[lo.repeat_interleave(cnt) + torch.arange(i.numel(), device=pos.device)
                      - first.repeat_interleave(cnt)]
            d = pos[i] - pos[j]
            d -= torch.round(d)
            r2 = (d * d).sum(-1)
            ok = (r2 < h[i] ** 2) & (i != j)
            yield i[ok], j[ok], d[ok], torch.sqrt(r2[ok])


def exact(case, seed):
    if case["mode"] != "fixed" or case["n"] > 400_000:
        return None      # a solved h is any h within the tolerance; larger sets take too long
    pos, h32, m32, u32, v32, _ = _particles(case, seed)
    h, m, u, v = h32.double(), m32.double(), u32.double(), v32.double()
    n = h.numel()
    zero = torch.zeros(n, dtype=torch.float64, device="cuda")
    sf, sg, sw, sq, cnt = (zero.clone() for _ in range(5))
    parts = [tuple(t) for t in _pairs(pos, h)]
    for i, j, _, r in parts:
        q = r / h[i]
        s = torch.clamp(0.5 - q, min=0.0)
        f = 2.0 * (1.0 - q) ** 3 - 8.0 * s ** 3
        qf = q * (24.0 * s ** 2 - 6.0 * (1.0 - q) ** 2)
        for acc, t in ((sf, m[j] * f), (sg, m[j] * (3.0 * f + qf)), (sw, f), (sq, qf), (cnt, torch.ones_like(f))):
            acc.index_add_(0, i, t)
    norm = 8.0 / math.pi / h ** 3
    rho, drho = norm * (m + sf), -norm / h * (3.0 * m + sg)
    nw, dnw = 32.0 / 3.0 * (1.0 + sw), -32.0 / 3.0 / h * sq
    A = (GAMMA - 1.0) * u / rho / (1.0 + h / (3.0 * rho) * drho)
    c = torch.sqrt(GAMMA * (GAMMA - 1.0) * u)
    acc = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    du, S, vs, nf = (zero.clone() for _ in range(4))

    def slope(r, k):             # (dW/dr) / r of the cubic spline with support h_k
        q = r / h[k]
        w = torch.where(q < 0.5, 18.0 * q - 12.0, torch.where(q < 1.0, -6.0 * (1.0 - q) ** 2 / q, 0.0))
        return 8.0 / math.pi / h[k] ** 5 * w

    for i, j, d, r in parts:
        back = r >= h[j]         # j's own support does not reach i: the pair counts for j too
        for a, b, e in ((i, j, d), (j[back], i[back], -d[back])):
            rr = r if a is i else r[back]
            ki, kj = slope(rr, a), slope(rr, b)
            vx = ((v[a] - v[b]) * e).sum(-1)
            w = torch.clamp(vx / rr, max=0.0)
            sig = c[a] + c[b] - 3.0 * w
            visc = -ALPHA * sig * w / (rho[a] + rho[b])
            kbar = 0.5 * (ki + kj)
            ms = m[b] * (A[a] * ki + A[b] * kj + visc * kbar)
            acc.index_add_(0, a, -ms[:, None] * e)
            du.index_add_(0, a, m[b] * vx * (A[a] * ki + 0.5 * visc * kbar))
            S.index_add_(0, a, ms.abs() * rr)
            nf.index_add_(0, a, torch.ones_like(rr))
            vs.scatter_reduce_(0, a, sig, "amax")
    sums = torch.stack([*(m[:, None] * acc).sum(0), (m * ((v * acc).sum(-1) + du)).sum(), (m * S).sum(), cnt.sum(),
                        nf.sum(), zero.sum()])
    got = {"rho": rho, "drho_dh": drho, "nw": nw, "dnw_dh": dnw, "nngb": None, "h": h, "f_ax": acc[:, 0],
           "f_ay": acc[:, 1], "f_az": acc[:, 2], "f_dudt": du, "f_vsig": vs, "f_S": S, "f_nforce": None, "f_sums": sums}
    return {**got, "hash": None, "f_hash": None} if case["hash"] else got
