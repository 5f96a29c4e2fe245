"""Scratch that a context holds after a call, per particle or site: the builders
need these bytes whatever launches their levels take, and a call near the
device's memory is admitted or refused by them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 400000


# few, large leaves: what counts is the scratch that goes with the particles
@pytest.mark.parametrize("what,most", [("octree", 90), ("kd", 537), ("voronoi", 199)])
def test_scratch_per_particle(what, most):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: scratch", what, flush=True)
    pos = np.random.default_rng(1).random((N, 3))
    ctx = pkg.Context(0)
    if what == "voronoi":
        pkg.build_voronoi(ctx, pos, n_lloyd=1)[0].free()
    else:
        kw = dict(leaf_max=200) if what == "octree" else dict(leaf_split=200, tree="kd")
        pkg.build_pseudo_particles(ctx, pos, np.full(N, 0.016), np.full(N, 1 / N), [[0.5, 0.5, 0.5]], **kw)
    torch.cuda.synchronize()
    held = ctx.workspace_info()["held"]
    ctx.close()
    print(f"   {held / N:.1f} bytes each", flush=True)
    assert held <= most * N
