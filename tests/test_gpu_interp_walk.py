"""The shared walk of the per-particle interpolation against the oracle where
its wavefronts go wrong first: last wavefronts of one to 63 particles, entry
counts around the hierarchy's groups of 16 and levels, 1 to 9 components (one
pass holds four), owners at random, so that the particles of a wavefront do
not lie within their entries' spheres, and smoothing lengths over 3.5 decades.

The same binary64 terms are summed in another order: fewer than 70,000 terms
of one sign, whose rounding stays under 70,000 2^-53 = 8e-12 at the worst and
sqrt of that factor, 3e-14, in practice; values agree within 1e-12 times the
largest entry value, as for the whole path."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,ne,comps", [
    (1, 1, 1), (63, 15, 2), (64, 16, 3), (65, 17, 4), (1000, 255, 5), (1001, 257, 9), (4097, 4096, 1), (4097, 4113, 8),
    (20001, 70001, 3),
])
def test_walk_matches_oracle(oracle, n, ne, comps):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: interpolation walk", n, ne, comps, flush=True)
    g = np.random.default_rng(n + ne)
    pos, ex = g.random((n, 3)), g.random((ne, 3))
    eh = 10.0 ** g.uniform(-4.0, -0.5, ne)
    ek = (g.random(ne) < 0.7).astype(np.int32)
    owner = g.integers(0, ne, n)
    values = g.normal(size=(ne, comps))
    ctx = pkg.Context(0)
    mixed = dict(xyz=torch.tensor(ex, device="cuda"), h=torch.tensor(eh, device="cuda"),
                 kind=torch.tensor(ek, device="cuda"), owner=torch.tensor(owner, device="cuda"))
    got = pkg.interpolate_to_particles(ctx, pos, mixed, values).cpu().numpy()
    want = oracle.interpolate(pos, owner, ex, eh, ek, values)
    ctx.close()
    real = ek[owner] == 0
    assert np.array_equal(got[real], want[real])
    assert np.abs(got - want).max() <= 1e-12 * np.abs(values).max()
