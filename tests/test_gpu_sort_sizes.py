"""The radix sorts and scans behind the builders and the transpose at the sizes
where their launches change: one workgroup (4,096 items), tiles of 2,048,
tiles that add up themselves (64 of them), a scan's block sums.  The octree
builder sorts 63-bit keys, and its entries are the oracle's exactly; the
particle-major copy is a stable sort of the pairs, and the inverse mapping of
the cell index replayed in numpy in the stated order is equal bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", params=[0, 16 << 30], ids=["free", "capped"])
def ctx(request):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = pkg.Context(0, workspace_bytes=request.param)
    yield c
    c.close()


@pytest.mark.parametrize("n", [1, 2, 65, 1024, 1025, 3073, 4095, 4096, 4097, 6143, 131072, 131073])
def test_octree_sort(ctx, n, oracle):
    import paper_2410_15227_amd as pkg
    print("case:", n, flush=True)
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3)) * np.where(rng.random(n) < 0.5, 1.0, 0.1)[:, None]
    m, h = np.full(n, 1.0 / n), np.full(n, 0.6 / max(n, 8) ** (1 / 3))
    src = [[0.05, 0.05, 0.05]]
    want = oracle.pseudo_build(pos, m, h, np.array(src), r_part=0.1, theta=0.5)
    got = pkg.build_pseudo_particles(ctx, pos, h, m, src, r_part=0.1, theta=0.5)
    assert np.array_equal(got["owner"].cpu().numpy(), want["owner"])
    assert np.array_equal(got["kind"].cpu().numpy(), want["kind"])
    assert np.array_equal(got["xyz"].cpu().numpy()[want["kind"] == 0], want["pos"][want["kind"] == 0])


@pytest.mark.parametrize("n", [3, 257, 1025, 2049])
def test_transpose_order(ctx, n, workloads):
    import paper_2410_15227_amd as pkg
    print("case:", n, flush=True)
    pos, m, h, _ = workloads.make_cloud("uniform", n, seed=n)
    dt = ctx.upload(workloads.voronoi(pos))
    res = pkg.map_particles_to_cells(ctx, dt, pos, h, m, keep_pairs=True)
    off, part, w = (a.cpu().numpy() for a in res.pairs.export())
    q = np.arange(n, dtype=np.float64) + 1.0
    got = pkg.map_cells_to_particles(ctx, res.pairs, q).cpu().numpy()
    cov = res.coverage.cpu().numpy()
    cell = np.repeat(np.arange(n), np.diff(off))
    order = np.argsort(part, kind="stable")
    cell, w, start = cell[order], w[order], np.searchsorted(part[order], np.arange(n + 1))
    for i in range(n):
        t = w[start[i]:start[i + 1]] * q[cell[start[i]:start[i + 1]]]
        lanes = [0.0] * 16
        for j, v in enumerate(t):
            lanes[j % 16] += v
        for o in (8, 4, 2, 1):
            lanes = [lanes[k] + lanes[k ^ o] for k in range(16)]
        assert got[i] == (lanes[0] / cov[i] if cov[i] > 0 else 0.0)
    res.pairs.free()
    dt.free()
