"""The binary64 edge kernel against the one-lane binary64 kernel (the path of
a context with a workspace cap), which evaluates the same closed form with
the math library: every weight within 1e-12 (the binary64 path's bar), where
the edge kernel's own limits lie -- more than 64 faces or 256 candidate edges
a pair, more face records than a wave holds, supports far smaller and far
larger than the cells, particles on faces, edges and vertices, chunks that
end within a cell."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def prism(sides, z0, z1, n):
    """A prism over a regular polygon about (0.5, 0.5), split into n cells along z."""
    a = 2.0 * np.pi * np.arange(sides) / sides
    ring = 0.5 + 0.4 * np.stack([np.cos(a), np.sin(a)], axis=1)
    gens, cells = [], []
    zs = np.linspace(z0, z1, n + 1)
    for lo, hi in zip(zs[:-1], zs[1:]):
        bot = np.column_stack([ring, np.full(sides, lo)])
        top = np.column_stack([ring, np.full(sides, hi)])
        k = np.arange(sides)
        j = (k + 1) % sides
        cells.append([bot[::-1], top] + [np.array([bot[p], bot[q], top[q], top[p]]) for p, q in zip(k, j)])
        gens.append([0.5, 0.5, 0.5 * (lo + hi)])
    return np.array(gens), cells


def case(name, workloads):
    rng = np.random.default_rng(77)
    if name.startswith("prism"):
        sides, n, h = {"prism70": (70, 2, 0.3), "prism60": (60, 3, 0.5), "prism40": (40, 3, 0.6)}[name]
        tess = workloads.tess_from_cells(*prism(sides, 0.0, 1.0, n))
        pos = rng.random((333, 3))
        return tess, pos, np.full(333, h)
    pos, m, h, _ = workloads.make_cloud("turbulent", 700, seed=6)
    tess = workloads.voronoi(pos)
    if name == "large_h":
        h = h * 6.0
    elif name == "small_h":
        h = h * 1e-3
    elif name == "on_grid":  # vertices, edge midpoints and face vertex means as particles
        v = tess.vertices[tess.face_vtx.astype(np.int64)]
        o = tess.face_vtx_off[:-1]
        pos = np.concatenate([v[o[:200]], 0.5 * (v[o[:200]] + v[o[:200] + 1]),
                              np.add.reduceat(v, o)[:200] / np.diff(tess.face_vtx_off)[:200, None], pos])
        h = np.resize(h, len(pos))
    return tess, pos, h


@pytest.mark.parametrize("name", ["prism70", "prism60", "prism40", "large_h", "small_h", "on_grid"])
def test_edge_kernel_matches_one_lane_kernel(name, workloads):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case:", name, flush=True)
    tess, pos, h = case(name, workloads)
    m = np.full(len(pos), 1.0 / len(pos))
    w = []
    for cap in (0, 8 << 30):
        ctx = pkg.Context(0, workspace_bytes=cap)
        dt = ctx.upload(tess)
        res = pkg.map_particles_to_cells(ctx, dt, pos, h, m, precision="fp64", keep_pairs=True)
        off, part, wt = res.pairs.export()
        w.append((off.cpu().numpy(), part.cpu().numpy(), wt.cpu().numpy()))
        res.pairs.free()
        dt.free()
        ctx.close()
    assert np.array_equal(w[0][0], w[1][0]) and np.array_equal(w[0][1], w[1][1])
    assert np.max(np.abs(w[0][2] - w[1][2])) < 1e-12
