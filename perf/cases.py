"""Measured cases of the mapping, the grid builder and the pseudo-particle
builder, each through the package's public entry points.

Every case names a kind of call and its sizes:

  map      forward mapping with its pair list kept, then the inverse mapping
           (one hydrodynamics timestep on a resident grid)
  inverse  inverse mapping of several components from a kept pair list
  voronoi  the grid of new sites with its Lloyd iterations, and its cell info
  pseudo   pseudo-particles of a cloud around one source (octree or k-d tree)
  interp   per-particle values from a mixed set
  batch    a planned batch of independent mappings, one graph launch a step
  step     the whole pseudo-particle timestep: build, grid of the mixed set,
           forward and inverse mapping, values of every particle
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2410_15227_amd as pkg
from paper_2410_15227_amd import workloads

R_PART, THETA, H_FACT = 0.2, 0.5, 1.2  # the walk of the 1M-particle pseudo workload

_context = None


def _ctx():
    """The library context a program keeps for all its calls."""
    global _context
    if _context is None:
        _context = pkg.Context(0)
    return _context


def listed():
    return [
        # the smallest mapping anyone runs: a test box; launches and latency
        dict(name="map_512", kind="map", n=512, cloud="uniform", precision="mixed", normalize=False, comps=1),
        # the binary64 reference box of 4,096 particles
        dict(name="map_4096_fp64", kind="map", n=4096, cloud="uniform", precision="fp64", normalize=False, comps=1),
        # an ordinary odd-sized cloud with conserved mass and three ionic fractions carried back
        dict(name="map_30011_norm", kind="map", n=30011, cloud="turbulent", precision="mixed", normalize=True, comps=3),
        # a turbulent cloud in binary64 throughout, as when a mixed result is to be checked
        dict(name="map_65521_fp64", kind="map", n=65521, cloud="turbulent", precision="fp64", normalize=False, comps=1),
        # the benchmark's timestep: 262,144 particles of a turbulent cloud
        dict(name="map_262144", kind="map", n=262144, cloud="turbulent", precision="mixed", normalize=False, comps=1),
        # several fields carried back from one forward mapping
        dict(name="inverse_100003", kind="inverse", n=100003, cloud="turbulent", comps=5),
        # regularised grid of new sites (five Lloyd iterations)
        dict(name="voronoi_131071", kind="voronoi", n=131071, cloud="turbulent", lloyd=5),
        # pseudo-particles of a million-particle cloud, octree
        dict(name="pseudo_1048576", kind="pseudo", n=1048576, tree="octree"),
        # the same from the k-d tree, on a smaller odd-sized cloud
        dict(name="pseudo_kd_262139", kind="pseudo", n=262139, tree="kd"),
        # a million particles' values from their mixed set
        dict(name="interp_1048576", kind="interp", n=1048576, comps=3),
        # eight small mappings of uneven size as one captured step
        dict(name="batch_8", kind="batch", count=8, lo=11.0, hi=15.0),
        # the whole timestep with pseudo-particles
        dict(name="step_200003", kind="step", n=200003, lloyd=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["map", "map", "map", "inverse", "voronoi", "pseudo", "interp", "batch", "step"])
    cloud = rng.choice(["uniform", "turbulent"])
    if kind == "map":
        precision = rng.choice(["mixed", "mixed", "fp64"])
        n = _log_int(rng, 300, 200000 if precision == "mixed" else 65000)
        return dict(kind=kind, n=n, cloud=cloud, precision=precision, normalize=rng.random() < 0.3,
                    comps=rng.choice([1, 1, 3]))
    if kind == "inverse":
        return dict(kind=kind, n=_log_int(rng, 1000, 150000), cloud=cloud, comps=rng.randint(1, 8))
    if kind == "voronoi":
        return dict(kind=kind, n=_log_int(rng, 1000, 131000), cloud=cloud, lloyd=rng.choice([0, 1, 5]))
    if kind == "pseudo":
        return dict(kind=kind, n=_log_int(rng, 5000, 1000000), tree=rng.choice(["octree", "kd"]))
    if kind == "interp":
        return dict(kind=kind, n=_log_int(rng, 5000, 1000000), comps=rng.randint(1, 4))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(2, 10), lo=9.0, hi=rng.uniform(11.0, 15.0))
    return dict(kind=kind, n=_log_int(rng, 20000, 200000), lloyd=rng.choice([0, 5]))


# ------------------------------------------------------------------- inputs
def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def _cloud(case, seed):
    """Positions, masses and self-consistent smoothing lengths."""
    return workloads.make_cloud(case["cloud"], case["n"], seed)[:3]


def _source_cloud(n, seed):
    """A turbulent cloud with smoothing lengths from its local number density
    (counted on a grid), and one source at the densest place."""
    pos = workloads.turbulent_cloud(n, seed, grid=128 if n > 100000 else 64)
    g = max(4, int(round((n / 16.0) ** (1.0 / 3.0))))
    at = np.minimum((pos * g).astype(np.int64), g - 1)
    key = (at[:, 0] * g + at[:, 1]) * g + at[:, 2]
    count = np.bincount(key, minlength=g ** 3)[key]
    h = H_FACT * np.cbrt(1.0 / (count * float(g) ** 3))
    return pos, np.full(n, 1.0 / n), h, pos[int(np.argmax(count))][None, :].copy()


def _fields(gen, comps):
    """Smooth cell fields in [0, 1], as ionic fractions are."""
    x = gen[:, :1] * (3.0 + np.arange(comps)) + gen[:, 1:2]
    f = 0.5 + 0.5 * np.sin(2.0 * np.pi * x)
    return f[:, 0] if comps == 1 else f


def _batch_mix(case, seed):
    """Clouds of sizes spread over the logarithm of the case's range."""
    out = []
    for k in range(case["count"]):
        n = int(round(2.0 ** (case["lo"] + (case["hi"] - case["lo"]) * (k + 0.37) / case["count"])))
        out.append(workloads.make_cloud("turbulent" if k % 2 else "uniform", n, seed + 7919 * k + 1)[:3])
    return out


def _ionisation(sites, source):
    """A Stroemgren-like sphere about the source, on the device."""
    r = torch.linalg.norm(sites - source, dim=1)
    return 0.5 * (1.0 + torch.tanh((r - 0.25) / 0.02))


def prepare(case, seed):
    ctx, kind = _ctx(), case["kind"]
    s = dict(case=case, ctx=ctx)
    if kind in ("map", "inverse"):
        pos, m, h = _cloud(case, seed)
        tess = workloads.voronoi(pos)
        s.update(grid=ctx.upload(tess), x=_dev(pos), h=_dev(h), m=_dev(m), q=_dev(_fields(pos, case["comps"])))
        if kind == "inverse":
            s["pairs"] = pkg.map_particles_to_cells(ctx, s["grid"], s["x"], s["h"], s["m"], keep_pairs=True).pairs
    elif kind == "voronoi":
        make = workloads.turbulent_cloud if case["cloud"] == "turbulent" else workloads.uniform_cloud
        s["x"] = _dev(make(case["n"], seed))
    elif kind == "batch":
        mix = _batch_mix(case, seed)
        grids = [ctx.upload(workloads.voronoi(pos)) for pos, _, _ in mix]
        s["plan"] = pkg.BatchPlan(ctx, grids, [_dev(p) for p, _, _ in mix], [_dev(h) for _, _, h in mix],
                                  [_dev(m) for _, m, _ in mix])
    else:
        pos, m, h, src = _source_cloud(case["n"], seed)
        s.update(x=_dev(pos), h=_dev(h), m=_dev(m), src=src)
        if kind == "interp":
            s["set"] = _pseudo(s)
            k = np.arange(case["comps"])
            e = s["set"]["xyz"][:, :1] * _dev(3.0 + k) + s["set"]["xyz"][:, 1:2]
            s["values"] = 0.5 + 0.5 * torch.sin(2.0 * math.pi * e)
        elif kind == "step":
            s["src_dev"] = _dev(src)
    return s


def _pseudo(s):
    return pkg.build_pseudo_particles(s["ctx"], s["x"], s["h"], s["m"], s["src"], r_part=R_PART, theta=THETA,
                                      h_fact=H_FACT, tree=s["case"].get("tree", "octree"))


def _kept(t, n):
    """t in a buffer of n rows, as a program holds what changes its length from step to step."""
    out = t.new_zeros((n, *t.shape[1:]))
    out[:len(t)] = t
    return out


# --------------------------------------------------------------------- pass
def run(s):
    ctx, case = s["ctx"], s["case"]
    kind = case["kind"]
    if kind == "map":
        r = pkg.map_particles_to_cells(ctx, s["grid"], s["x"], s["h"], s["m"], precision=case["precision"],
                                       normalize=case["normalize"], keep_pairs=True)
        q = pkg.map_cells_to_particles(ctx, r.pairs, s["q"])
        r.pairs.free()
        return dict(mass=r.mass, density=r.density, coverage=r.coverage, values=q)
    if kind == "inverse":
        return dict(values=pkg.map_cells_to_particles(ctx, s["pairs"], s["q"]))
    if kind == "voronoi":
        grid, sites = pkg.build_voronoi(ctx, s["x"], n_lloyd=case["lloyd"])
        volume, radius = grid.cell_info()
        grid.free()
        return dict(sites=sites, volume=volume, radius=radius)
    if kind == "pseudo":
        ps, n = _pseudo(s), case["n"]
        return {k: v if k in ("owner", "stats") else _kept(v, n) for k, v in ps.items()}
    if kind == "interp":
        return dict(values=pkg.interpolate_to_particles(ctx, s["x"], s["set"], s["values"]))
    if kind == "batch":
        s["plan"].run()
        return dict(mass=s["plan"].mass, density=s["plan"].density, coverage=s["plan"].coverage)
    ps = _pseudo(s)
    grid, sites = pkg.build_voronoi(ctx, ps["xyz"], n_lloyd=case["lloyd"])
    r = pkg.map_particles_to_cells(ctx, grid, ps["xyz"], ps["h"], ps["m"], keep_pairs=True)
    q = pkg.map_cells_to_particles(ctx, r.pairs, _ionisation(sites, s["src_dev"]))
    values = pkg.interpolate_to_particles(ctx, s["x"], ps, q)
    r.pairs.free()
    grid.free()
    n = case["n"]
    return dict(entries=_kept(ps["xyz"], n), h=_kept(ps["h"], n), sites=_kept(sites, n), mass=_kept(r.mass, n),
                density=_kept(r.density, n), entry_values=_kept(q, n), values=values)


# --------------------------------------------------------------------- work
CELL_BYTES = 24 + 7 * 24 + 16 * 12 + 80 * 4  # generator, vertices, face offsets and neighbours, vertex indices


def _pairs(n, cloud):
    """Candidate pairs of n particles on the grid of their own positions:
    about 158 a particle in a turbulent cloud, 144 in a uniform one, fewer
    where the support of a small box's particles passes its walls."""
    return n * (158 if cloud == "turbulent" else 144) / (1.0 + 1.7 * n ** (-1.0 / 3.0))


def work(case):
    kind = case["kind"]
    if kind == "map":
        p, n, k = _pairs(case["n"], case["cloud"]), case["n"], case["comps"]
        return dict(bytes=n * (40 + 24 + 16 * k + CELL_BYTES) + 24 * p, flops=p * (2512 + 4 + 2 * k))
    if kind == "inverse":
        p, k = _pairs(case["n"], case["cloud"]), case["comps"]
        return dict(bytes=12 * p + 16 * k * case["n"], flops=2 * k * p)
    if kind == "voronoi":
        # per cell and construction: 16 cuts of about 25 vertices (8 operations each), 80 new vertices (60 each)
        return dict(bytes=case["n"] * (24 + 24 + 12 + CELL_BYTES), flops=case["n"] * (case["lloyd"] + 1) * 8000)
    if kind == "pseudo":
        return dict(bytes=case["n"] * (40 + 8 + 0.16 * 68), flops=case["n"] * 20 * 8)
    if kind == "interp":
        n, k = case["n"], case["comps"]
        return dict(bytes=n * (24 + 8 + 8 * k) + 0.16 * n * (36 + 8 * k), flops=n * 60 * (20 + 2 * k))
    if kind == "batch":
        n = case["count"] * (2.0 ** case["hi"] - 2.0 ** case["lo"]) / ((case["hi"] - case["lo"]) * math.log(2.0))
        p = n * 140
        return dict(bytes=n * (40 + 24 + CELL_BYTES), flops=p * 2516)
    n = case["n"]
    e = 0.3 * n
    return dict(bytes=n * (40 + 8 + 32) + e * (68 + 48 + 2 * CELL_BYTES + 24 * 150),
                flops=n * (160 + 60 * 22) + e * (8000 * (case["lloyd"] + 1) + 150 * 2518))


# -------------------------------------------------- the same in plain binary64
def _planes(x, near):
    """Half-spaces n.r <= d about each site x: bisectors of its neighbours, then the walls of the unit box."""
    v = near - x[:, None]
    dist = torch.linalg.norm(v, dim=2, keepdim=True)
    eye = torch.eye(3, dtype=x.dtype, device=x.device).expand(len(x), 3, 3)
    return torch.cat([v / dist, -eye, eye], 1), torch.cat([0.5 * dist[..., 0], x, 1.0 - x], 1)


def _edges(sites):
    """Directed edges of the cells, each as seen from one of its two faces
    (counter-clockwise from outside): cell, face normal, face offset, ends,
    all about the cell's site, ordered by cell."""
    n, dev = len(sites), sites.device
    todo, k, parts = torch.arange(n, device=dev), min(48, n - 1), []
    while len(todo):
        again = []
        for at in torch.split(todo, max(1, int(1.2e8 / (k + 6) ** 3))):
            x = sites[at]
            d2 = sum((x[:, None, a] - sites[None, :, a]) ** 2 for a in range(3))
            near = torch.topk(d2, k + 1, dim=1, largest=False, sorted=True)
            N, d = _planes(x, sites[near.indices[:, 1:]])
            P = N.shape[1]
            u = torch.linalg.cross(N[:, :, None], N[:, None, :])
            u2 = (u * u).sum(3, keepdim=True).clamp_min(1e-300)
            p0 = (d[:, :, None, None] * torch.linalg.cross(N[:, None, :].expand_as(u), u)
                  + d[:, None, :, None] * torch.linalg.cross(u, N[:, :, None].expand_as(u))) / u2
            u = u / u2.sqrt()
            den = (u.reshape(len(x), P * P, 3) @ N.transpose(1, 2)).reshape(len(x), P, P, P)
            gap = d[:, None, None, :] - (p0.reshape(len(x), P * P, 3) @ N.transpose(1, 2)).reshape(len(x), P, P, P)
            i = torch.arange(P, device=dev)
            own = (i[:, None, None] == i) | (i[None, :, None] == i)
            inf = torch.tensor(math.inf, dtype=x.dtype, device=dev)
            t = gap / den
            hi = torch.where((den > 1e-13) & ~own, t, inf).amin(3)
            lo = torch.where((den < -1e-13) & ~own, t, -inf).amax(3)
            out = ((den.abs() <= 1e-13) & (gap < 0) & ~own).any(3) | (u2[..., 0] < 1e-24)
            c, a, b = torch.nonzero((hi > lo) & ~out, as_tuple=True)
            A = p0[c, a, b] + lo[c, a, b, None] * u[c, a, b]
            B = p0[c, a, b] + hi[c, a, b, None] * u[c, a, b]
            r2 = torch.zeros(len(x), dtype=x.dtype, device=dev)
            r2.scatter_reduce_(0, c, (A * A).sum(1), "amax")
            # no site further out can cut: it is beyond twice the cell's radius, or no vertex lies nearer to it
            sure = (near.values[:, -1] > 4.0 * r2) | (k == n - 1)
            ask = torch.nonzero(~sure[c])[:, 0]
            cut = torch.zeros(len(x), dtype=torch.bool, device=dev)
            for e in torch.split(ask, max(1, int(1e8 / n))):
                v = x[c[e]] + A[e]
                dv = sum((v[:, None, a] - sites[None, :, a]) ** 2 for a in range(3)).amin(1)
                cut[c[e][dv < (A[e] * A[e]).sum(1) * (1.0 - 1e-10)]] = True
            sure |= ~cut
            keep = sure[c]
            parts.append([v[keep] for v in (at[c], N[c, a], d[c, a], A, B)])
            again.append(at[~sure])
        todo, k = torch.cat(again), min(2 * k, n - 1)
    cell, nrm, d, A, B = (torch.cat(v) for v in zip(*parts))
    order = torch.argsort(cell, stable=True)
    return cell[order], nrm[order], d[order], A[order], B[order]


def _phi(q):
    """Integral of M(q) / q^2, M the mass of the M4 kernel within q smoothing lengths."""
    inner = q * q * (2.0 / 3.0 + q * q * (-0.3 + 0.1 * q))
    outer = q * q * (4.0 / 3.0 + q * (-1.0 + q * (0.3 - q / 30.0))) + 1.0 / (15.0 * q) - 0.2
    return torch.where(q < 1.0, inner, torch.where(q < 2.0, outer, 1.4 - 1.0 / q))


def _edge_terms(D, p, t0, t1, rule):
    """Flux of the kernel's field through the triangles (foot point, edge) of
    a plane at signed distance D, all in smoothing lengths: Gauss-Legendre
    along the edge between the places where it crosses q = 1 and q = 2."""
    z, wt = rule
    s2 = D * D + p * p
    k1, k2 = (1.0 - s2).clamp_min(0).sqrt(), (4.0 - s2).clamp_min(0).sqrt()
    knots = torch.stack([t0, -k2, -k1, k1, k2, t1], 1)
    knots = torch.minimum(torch.maximum(knots, t0[:, None]), t1[:, None])
    base, total = _phi(D.abs().clamp_min(1e-300))[:, None], torch.zeros_like(D)
    for j in range(5):
        a, half = knots[:, j, None], 0.5 * (knots[:, j + 1, None] - knots[:, j, None])
        t = a + half * (z + 1.0)
        tt = p[:, None] ** 2 + t * t
        f = (_phi((D[:, None] ** 2 + tt).sqrt()) - base) / tt.clamp_min(1e-300)
        total += (half * f * wt).sum(1)
    return D * p * total / (4.0 * math.pi)


def _weights(gen, x, h):
    """(cell, particle, weight) of every pair that can overlap, and the cell volumes."""
    cell, nrm, d, A, B = _edges(gen)
    C, dev = len(gen), gen.device
    first = torch.searchsorted(cell, torch.arange(C + 1, device=dev))
    r = torch.zeros(C, dtype=gen.dtype, device=dev)
    r.scatter_reduce_(0, cell, torch.linalg.norm(A, dim=1), "amax")
    u = torch.nn.functional.normalize(B - A, dim=1)
    out = torch.linalg.cross(u, nrm)
    volume = torch.zeros_like(r).index_add_(0, cell, d * (A * out).sum(1) * ((B - A) * u).sum(1) / 6.0)
    z, wt = np.polynomial.legendre.leggauss(16)
    rule = _dev(z), _dev(wt)
    found = []
    for at in torch.split(torch.arange(C, device=dev), max(1, int(2e8 / len(x)))):
        d2 = sum((gen[at, None, a] - x[None, :, a]) ** 2 for a in range(3))
        c, i = torch.nonzero(d2 < (r[at, None] + 2.0 * h[None, :]) ** 2, as_tuple=True)
        c = at[c]
        w = torch.zeros(len(c), dtype=x.dtype, device=dev)
        for part in torch.split(torch.arange(len(c), device=dev), 12000):
            cnt = (first[1:] - first[:-1])[c[part]]
            pair = torch.repeat_interleave(part, cnt)
            e = torch.arange(len(pair), device=dev) - torch.repeat_interleave(cnt.cumsum(0) - cnt - first[c[part]], cnt)
            rel, hp = x[i[pair]] - gen[c[pair]], h[i[pair]]
            D = (d[e] - (nrm[e] * rel).sum(1)) / hp
            p = (out[e] * (A[e] - rel)).sum(1) / hp
            t0, t1 = ((u[e] * (v[e] - rel)).sum(1) / hp for v in (A, B))
            w.index_add_(0, pair, _edge_terms(D, p, t0, t1, rule))
        found.append((c, i, w))
    return (*(torch.cat(v) for v in zip(*found)), volume)


def _mapped(pos, m, h, normalize=False, q=None):
    x, m, h = _dev(pos), _dev(m), _dev(h)
    c, i, w, volume = _weights(x, x, h)
    cover = torch.zeros_like(m).index_add_(0, i, w)
    mass = torch.zeros_like(m).index_add_(0, c, w * (m / cover if normalize else m)[i])
    r = dict(mass=mass, density=mass / volume, coverage=cover)
    if q is not None:
        v = _dev(q).reshape(len(x), -1)
        r["values"] = (torch.zeros_like(v).index_add_(0, i, w[:, None] * v[c]) / cover[:, None]).reshape(q.shape)
    return r


def _grid_info(sites, lloyd):
    for it in range(lloyd + 1):
        cell, nrm, d, A, B = _edges(sites)
        n = len(sites)
        # signed volume and first moment of the tetrahedra (site, foot point of the face, edge)
        foot = d[:, None] * nrm
        v = (nrm * torch.linalg.cross(A - foot, B - foot)).sum(1) * d / 6.0
        volume = torch.zeros(n, dtype=sites.dtype, device=sites.device).index_add_(0, cell, v)
        if it < lloyd:
            move = torch.zeros_like(sites).index_add_(0, cell, v[:, None] * (foot + A + B) / 4.0)
            sites = sites + move / volume[:, None]
    radius = torch.zeros_like(volume).scatter_reduce_(0, cell, torch.linalg.norm(A, dim=1), "amax")
    return dict(sites=sites, volume=volume, radius=radius.float())


def _interpolated(s):
    """Shepard interpolant over all entries for the members of pseudo-particles, the owner's value for the others."""
    e, v = s["set"], s["values"]
    out = v[e["owner"]].clone()
    member = torch.nonzero(e["kind"][e["owner"]] == 1)[:, 0]
    inv = 1.0 / e["h"]
    for at in torch.split(member, max(1, int(1.5e8 / len(inv)))):
        x = s["x"][at]
        q = (sum((x[:, None, a] - e["xyz"][None, :, a]) ** 2 for a in range(3))).sqrt_() * inv
        w = torch.where(q < 1.0, 1.0 + q * q * (0.75 * q - 1.5), 0.25 * (2.0 - q).clamp_min(0.0) ** 3)
        norm = w.sum(1, keepdim=True)
        out[at] = torch.where(norm > 0, (w @ v) / norm.clamp_min(1e-300), out[at])
    return dict(values=out)


def exact(case, seed):
    """What run returns, in plain binary64 torch: cells from all bisector
    half-spaces, the kernel integral by the divergence theorem with
    Gauss-Legendre along the edges.  None where that would take too long, and
    for the trees, whose outputs are the tree's own."""
    kind = case["kind"]
    if kind in ("map", "inverse") and case["n"] <= 70000:
        pos, m, h = _cloud(case, seed)
        r = _mapped(pos, m, h, case.get("normalize", False), _fields(pos, case["comps"]))
        return r if kind == "map" else dict(values=r["values"])
    if kind == "voronoi" and case["n"] * (case["lloyd"] + 1) <= 800000:
        return _grid_info(prepare(case, seed)["x"], case["lloyd"])
    if kind == "interp" and case["n"] <= 300000:
        return _interpolated(prepare(case, seed))
    if kind == "batch":
        mix = _batch_mix(case, seed)
        if sum(len(m) for _, m, _ in mix) <= 100000:
            r = [_mapped(*cloud) for cloud in mix]
            return {k: [v[k] for v in r] for k in ("mass", "density", "coverage")}
    return None
