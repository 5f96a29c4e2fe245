"""The shared faces' gifts reach the right pairs: mixed weights against the
binary64 path's, which evaluates every face from its own side.  Pairs per cell
around the gather's sizes (64 lanes, 256 pairs a window, bisected lists beyond
512) and a cell that takes more faces than are listed at a time (32).

A gift that is lost, doubled or given to another pair changes a weight by its
face's part of it, 1e-3 to 1; the paths differ by less than the mixed bar of
1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def hub_sites():
    """40 sites on a sphere, 60 beyond it and, last, its centre: every face of
    the centre's cell is evaluated by the other side."""
    g = np.random.default_rng(17)
    k = np.arange(40) + 0.5
    z, phi = 1.0 - 2.0 * k / 40, np.pi * (1.0 + 5.0 ** 0.5) * k
    r = np.sqrt(1.0 - z * z)
    shell = 0.5 + 0.25 * np.stack([r * np.cos(phi), r * np.sin(phi), z], axis=1)
    far = g.random((400, 3))
    far = far[np.linalg.norm(far - 0.5, axis=1) > 0.4][:60]
    return np.concatenate([shell, far, [[0.5, 0.5, 0.5]]])


@pytest.mark.parametrize("n,h", [(40, 0.05), (2500, 0.05), (4000, 0.1), (12000, 0.02), (30000, 0.1)])
def test_gifts_reach_their_pairs(n, h):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: gather", n, h, flush=True)
    ctx = pkg.Context(0)
    dt, _ = pkg.build_voronoi(ctx, hub_sites(), n_lloyd=0)
    tess = dt.export()
    faces = np.diff(tess.cell_face_off)
    assert faces[-1] > 32
    grid = pkg.DeviceTessellation(ctx, tess)
    assert grid.n_shared > 0
    g = np.random.default_rng(n)
    x, hh, m = g.random((n, 3)), np.full(n, h), g.uniform(0.5, 1.5, n)
    w = {}
    for precision in ("fp64", "mixed"):
        r = pkg.map_particles_to_cells(ctx, grid, x, hh, m, precision=precision, keep_pairs=True)
        off, part, w[precision] = (t.cpu().numpy() for t in r.pairs.export())
        r.pairs.free()
    print("   faces", faces[-1], "pairs per cell", np.diff(off).min(), np.diff(off).max(), flush=True)
    assert np.abs(w["mixed"] - w["fp64"]).max() < 1e-5
    ctx.close()
