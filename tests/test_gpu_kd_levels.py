"""k-d builds whose levels are launched in runs against the oracle: trees
shallower and deeper than the first run, levels on both sides of the
one-workgroup split (1024 nodes), depth limits at the ends of runs, and the
one-level runs of a context with a workspace cap.  The emitted set is
identical, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def cloud(name, n):
    g = np.random.default_rng(n)
    x = g.random((n, 3))
    if name == "deep":  # half of what is left in each halving of the distance to a corner
        x *= 0.5 ** g.geometric(0.5, n)[:, None].astype(np.float64)
    elif name == "point":  # nothing to split
        x[:] = 0.37
    return x


@pytest.mark.parametrize("cap", [0, 1 << 30])
@pytest.mark.parametrize("name,n,leaf_split,max_depth", [
    ("uniform", 1, 8, 40), ("uniform", 2, 2, 40), ("uniform", 131, 2, 62), ("uniform", 4099, 8, 0),
    ("uniform", 4099, 8, 9), ("uniform", 4099, 8, 10), ("uniform", 20011, 2, 40), ("deep", 20011, 8, 40),
    ("deep", 5003, 2, 14), ("point", 3001, 8, 40),
])
def test_levels_match_oracle(cap, name, n, leaf_split, max_depth, oracle):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: k-d levels", cap, name, n, leaf_split, max_depth, flush=True)
    x = cloud(name, n)
    m, h = np.random.default_rng(1).uniform(0.5, 1.5, n), np.full(n, 0.02)
    kw = dict(r_part=0.1, theta=0.6, leaf_split=leaf_split, max_depth=max_depth)
    src = np.array([[0.9, 0.9, 0.9]])
    ref = oracle.kd_build(x, m, h, src, **kw)
    ctx = pkg.Context(0, workspace_bytes=cap)
    got = pkg.build_pseudo_particles(ctx, x, h, m, src, tree="kd", **kw)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in got.items() if k != "stats"}
    ctx.close()
    for a, b in (("kind", "kind"), ("first", "first"), ("count", "count"), ("level", "level"), ("owner", "owner"),
                 ("xyz", "pos"), ("m", "mass"), ("s", "s")):
        assert np.array_equal(g[a], ref[b]), a
    assert np.array_equal(g["label"].view(np.uint64), ref["label"])
    assert got["stats"]["n_nodes"] == ref["stats"]["n_nodes"]
