"""Grids in blocks that earlier grids gave back: the same cells, bit for bit,
as in fresh memory, whichever context frees them and with the pool off; a
grid may outlive the context that made it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def build(ctx, n):
    import paper_2410_15227_amd as pkg
    dt, _ = pkg.build_voronoi(ctx, np.random.default_rng(n).random((n, 3)), n_lloyd=1)
    t = dt.export()
    vol, rad = (a.cpu().numpy() for a in dt.cell_info())
    return dt, [t.generators, t.vertices, t.cell_face_off, t.face_vtx_off, t.face_vtx, t.face_nbr, vol, rad]


@pytest.mark.parametrize("limit", [None, 0, 1 << 20])
def test_reused_blocks_hold_the_same_cells(limit):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: grid pool", limit, flush=True)
    sizes = (900, 1200, 17, 1300, 700, 1200)
    want = {}
    for n in set(sizes):
        fresh = pkg.Context(0)
        dt, want[n] = build(fresh, n)
        dt.free()
        fresh.close()
    ctx, other = pkg.Context(0), pkg.Context(0)
    if limit is not None:
        ctx.set_pool_limit(limit)
    kept = []
    for k, n in enumerate(sizes):
        dt, got = build(ctx, n)
        for a, b in zip(got, want[n]):
            assert np.array_equal(a, b), n
        if k % 3 == 2:
            kept.append((dt, n))  # lives on while its maker's other blocks are reused
        elif k % 3 == 1:
            dt.ctx = other
            dt.free()
        else:
            dt.free()
    ctx.close()
    for dt, n in kept:  # outlives its maker
        dt.ctx = other
        vol, _ = dt.cell_info()
        assert np.array_equal(vol.cpu().numpy(), want[n][6])
        dt.free()
    other.close()
