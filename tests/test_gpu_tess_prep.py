"""Face, edge and cell preparation against the oracle and closed forms: rows of
N-gon prisms whose cells fit a workgroup's LDS (N up to 21), exceed its slots
(22), fill its faces exactly (30) and exceed them (40), with face orientations
at random and a last workgroup of one cell.

Volumes and radii are the closed forms' to rounding (1e-13); binary64 weights
agree with the oracle's within 1e-12, the bar of that path."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def prisms(n_cells, N, seed):
    """n_cells prisms over regular N-gons, along x, generation sites off centre."""
    from paper_2410_15227_amd.workloads import Tessellation
    g = np.random.default_rng(seed)
    a = 2.0 * np.pi * np.arange(N) / N
    ring = 0.04 * np.stack([np.cos(a), np.sin(a)], axis=1)
    gen, vert, cfo, fvo, fv = [], [], [0], [0], []
    for c in range(n_cells):
        o = np.array([0.08 + 0.09 * c, 0.5, 0.5])
        base = len(vert)
        for z in (-0.03, 0.03):
            vert += [o + [x, y, z] for x, y in ring]
        faces = [list(range(N)), list(range(N, 2 * N))]
        faces += [[k, (k + 1) % N, N + (k + 1) % N, N + k] for k in range(N)]
        for k in g.permutation(len(faces)):
            f = faces[k] if g.random() < 0.5 else faces[k][::-1]
            fv += [base + v for v in f]
            fvo.append(len(fv))
        cfo.append(len(fvo) - 1)
        gen.append(o + g.uniform(-0.01, 0.01, 3))
    vert = np.array(vert)
    return Tessellation(generators=np.array(gen), vertices=vert, cell_face_off=np.array(cfo, dtype=np.int64),
                        face_vtx_off=np.array(fvo, dtype=np.int64), face_vtx=np.array(fv, dtype=np.int32),
                        face_nbr=np.full(len(fvo) - 1, -1, dtype=np.int32), box_lo=np.zeros(3), box_hi=np.ones(3))


@pytest.mark.parametrize("n_cells,N", [(1, 3), (8, 4), (9, 21), (9, 22), (8, 30), (9, 40)])
def test_prisms(oracle, n_cells, N):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: tessellation preparation", n_cells, N, flush=True)
    t = prisms(n_cells, N, N)
    ctx = pkg.Context(0)
    dt = pkg.DeviceTessellation(ctx, t)
    vol, rad = (x.cpu().numpy() for x in dt.cell_info())
    want = 0.06 * 0.5 * N * 0.04 ** 2 * np.sin(2.0 * np.pi / N)
    assert np.abs(vol / want - 1.0).max() < 1e-13
    d = np.linalg.norm(t.vertices.reshape(n_cells, 2 * N, 3) - t.generators[:, None], axis=2).max(axis=1)
    assert np.abs(rad / d - 1.0).max() < 2.0 ** -23 and (rad.astype(np.float64) >= d * (1.0 - 1e-15)).all()
    g = np.random.default_rng(1)
    n = 150
    x = np.stack([g.uniform(0.03, 0.12 + 0.09 * n_cells, n) % 1.0, g.uniform(0.44, 0.56, n), g.uniform(0.45, 0.55, n)], axis=1)
    h, m = np.full(n, 0.02), np.ones(n)
    r = pkg.map_particles_to_cells(ctx, dt, x, h, m, precision="fp64", keep_pairs=True)
    off, part, w = (a.cpu().numpy() for a in r.pairs.export())
    roff, rpart, rw = oracle.pairs_weights(t, x, h)
    assert np.array_equal(off, roff) and np.array_equal(part, rpart)
    assert np.abs(w - rw).max() < 1e-12
    ctx.close()
