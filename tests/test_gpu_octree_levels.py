"""Octree builds whose levels are launched in runs against the oracle: trees
shallower and deeper than the first run, node arrays that have to grow inside
a run, depth limits, large leaves, and the one-level runs of a context with a
workspace cap.  The emitted set is identical, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cloud(name, n):
    g = np.random.default_rng(n)
    x = g.random((n, 3))
    if name == "deep":  # half of what is left in each halving of the distance to a corner
        x *= 0.5 ** g.geometric(0.5, n)[:, None].astype(np.float64)
    elif name == "pairs":  # chains of single children: more nodes than the arrays start with
        x = np.repeat(x[: n // 2], 2, axis=0)
        x[1::2] = np.nextafter(x[1::2], 0.0)
    return x


@pytest.mark.parametrize("cap", [0, 4 << 30])
@pytest.mark.parametrize("name,n,leaf_max,max_depth", [
    ("uniform", 1, 8, 21), ("uniform", 9, 8, 21), ("uniform", 4099, 8, 1), ("uniform", 4099, 8, 3),
    ("uniform", 33000, 8, 4), ("uniform", 20011, 1, 21), ("uniform", 5003, 600, 21), ("deep", 20011, 8, 21),
    ("pairs", 20000, 1, 21), ("pairs", 3000, 1, 9),
])
def test_levels_match_oracle(cap, name, n, leaf_max, max_depth, oracle):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: octree levels", cap, name, n, leaf_max, max_depth, flush=True)
    x = cloud(name, n)
    m, h = np.random.default_rng(1).uniform(0.5, 1.5, n), np.full(n, 0.02)
    kw = dict(r_part=0.1, theta=0.6, leaf_max=leaf_max, max_depth=max_depth)
    src = np.array([[0.9, 0.9, 0.9]])
    ref = oracle.pseudo_build(x, m, h, src, **kw)
    ctx = pkg.Context(0, workspace_bytes=cap)
    got = pkg.build_pseudo_particles(ctx, x, h, m, src, **kw)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in got.items() if k != "stats"}
    ctx.close()
    for a, b in (("kind", "kind"), ("first", "first"), ("count", "count"), ("owner", "owner"), ("xyz", "pos"),
                 ("m", "mass"), ("s", "s"), ("branch", "branch")):
        assert np.array_equal(g[a], ref[b]), a
    assert np.array_equal(g["label"].view(np.uint64), ref["label"])
    assert got["stats"]["n_nodes"] == ref["n_nodes"]
