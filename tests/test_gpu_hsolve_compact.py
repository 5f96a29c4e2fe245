"""Node h-solve of nodes far smaller than binary32 resolves near the corner of
the box (their squared distances or inverse lengths leave its range): branch
and h are the oracle's, whose sums are binary64.  Only the power function may
differ in the last bit, hence 1e-9 h0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U = 2.0 ** -74  # spacing of doubles below 2^-21, where the octree's smallest cells meet
P = 2.0 ** -21


# pair: a node on either side of x = 2^-21, 6 U apart, seen from between them;
# point: two particles 1e-38 apart, whose lengths have no binary32 inverse
@pytest.mark.parametrize("name,x,src,h_fact", [
    ("pair", [P - U, P - 3 * U, P + 2 * U, P + 6 * U], P, 0.8),
    ("point", [0.0, 1e-38], 0.7, 0.5),
    ("point", [0.0, 1e-40], 0.7, 0.5),
])
def test_compact_nodes_match_oracle(name, x, src, h_fact, oracle):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: compact", name, x, flush=True)
    far = np.random.default_rng(1).random((64 - len(x), 3)) * 0.5 + 0.4  # 64 in all: masses and their sums exact
    pos = np.concatenate([np.array([[v, 0.0, 0.0] for v in x]), far])
    m, h = np.full(len(pos), 1.0 / len(pos)), np.full(len(pos), 0.1)
    kw = dict(r_part=0.0, theta=0.6, leaf_max=1)
    want = oracle.pseudo_build(pos, m, h, [[src, 0.0, 0.0]], hfact=h_fact, bypass=1 << 30, **kw)
    ctx = pkg.Context(0)
    got = pkg.build_pseudo_particles(ctx, pos, h, m, [[src, 0.0, 0.0]], h_fact=h_fact, bypass_threshold=1 << 30, **kw)
    torch.cuda.synchronize()
    ps = want["kind"] == 1
    small = ps & (want["s"] < 1e-20)
    g = {k: v.cpu().numpy() for k, v in got.items() if k != "stats"}
    ctx.close()
    assert small.sum() == (2 if name == "pair" else 1) and (want["branch"][small] > 0).all()
    assert np.array_equal(g["branch"], want["branch"])
    assert np.array_equal(g["s"], want["s"])
    assert (np.abs(g["h"][ps] - want["h"][ps]) <= 1e-9 * 2 * h_fact * want["s"][ps]).all()
