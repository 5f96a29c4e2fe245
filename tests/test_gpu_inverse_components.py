"""Inverse mapping of 1 to 17 components at once: each component's sums are its
own, in the stated order, so every column equals the one-component call's
result bit for bit (a pass takes up to eight components: 8, 9 and 17 are its
edges), and a particle that no cell covers gets 0 in all."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 17])
def test_columns_equal_single_calls(k, workloads):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case:", k, flush=True)
    ctx = pkg.Context(0)
    pos, m, h, _ = workloads.make_cloud("turbulent", 777, seed=8)
    dt = ctx.upload(workloads.voronoi(pos))
    x = np.concatenate([pos, [[3.0, 3.0, 3.0]]])  # outside the grid: no coverage
    res = pkg.map_particles_to_cells(ctx, dt, x, np.append(h, 0.01), np.append(m, 1.0), keep_pairs=True)
    q = torch.tensor(np.random.default_rng(k).standard_normal((777, k)), device="cuda")
    got = pkg.map_cells_to_particles(ctx, res.pairs, q)
    assert got.shape == (778, k) and bool((got[-1] == 0).all())
    for r in range(k):
        assert torch.equal(got[:, r], pkg.map_cells_to_particles(ctx, res.pairs, q[:, r].contiguous()))
    res.pairs.free()
    dt.free()
    ctx.close()
