"""Node h-solve with many units in reach: the workgroup-per-node Newton kernel
and the bracket's bounds against the one-wave sums, which a context with a
workspace cap keeps to.  Both add in unit order, so every array is equal bit
for bit; the units lie around the sizes where the kernels change over (96
tiles of 64 units in reach, 2048 tiles a workgroup holds)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def both():
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    free, capped = pkg.Context(0), pkg.Context(0, workspace_bytes=4 << 30)
    yield free, capped
    free.close()
    capped.close()


# corner: far nodes whose first step already reaches every unit; centre: nodes of all sizes
@pytest.mark.parametrize("n,kind,source,r_part,least,most", [
    (5003, "uniform", 0.02, 0.9, 1, 96 * 64),               # too few units for the wide kernel
    (27011, "uniform", 0.02, 1.1, 96 * 64 + 1, 120 * 64),   # just above the line
    (60013, "turbulent", 0.5, 0.5, 96 * 64 + 1, 60013),
    (300007, "turbulent", 0.3, 0.4, 96 * 64 + 1, 300007),
    (400009, "uniform", 0.02, 1.1, 2048 * 64 + 1, 400009),  # more tiles than a workgroup holds
])
def test_wide_sums_are_the_one_wave_sums(both, workloads, n, kind, source, r_part, least, most):
    import paper_2410_15227_amd as pkg
    print("case: h-solve", n, kind, source, r_part, flush=True)
    pos, m, h, rho = workloads.make_cloud(kind, n, seed=n)
    src = np.array([[source] * 3])
    free, capped = (pkg.build_pseudo_particles(c, pos, h, m, src, r_part=r_part, theta=0.6, bypass_threshold=1 << 30)
                    for c in both)
    torch.cuda.synchronize()
    print("  ", free["stats"], flush=True)
    assert least <= free["stats"]["n_units"] <= most and free["stats"]["n_pseudo"] > 0
    assert free["stats"] == capped["stats"]
    for k in free:
        if k != "stats":
            assert torch.equal(free[k], capped[k]), k


# nodes that the bracket solves: their signs from boxes, binary32 and binary64
# sums are those of the unit-order sums, so that branch and h are the oracle's
# (only its power function may differ in the last bit, hence 1e-9 h0)
@pytest.mark.parametrize("n,kind,source,r_part", [
    (63, "uniform", 0.5, 0.05), (5003, "turbulent", 0.5, 0.1), (27011, "uniform", 0.02, 1.1),
    (60013, "turbulent", 0.5, 0.5),
])
def test_bracket_matches_oracle(both, oracle, workloads, n, kind, source, r_part):
    import paper_2410_15227_amd as pkg
    print("case: h-solve bracket", n, kind, source, r_part, flush=True)
    pos, m, h, rho = workloads.make_cloud(kind, n, seed=n)
    src = np.array([[source] * 3])
    want = oracle.pseudo_build(pos, m, h, src, r_part=r_part, theta=0.6, bypass=1 << 30)
    got = pkg.build_pseudo_particles(both[0], pos, h, m, src, r_part=r_part, theta=0.6, bypass_threshold=1 << 30)
    ps = want["kind"] == 1
    branch = got["branch"].cpu().numpy()
    print("   branches", np.bincount(branch[ps], minlength=4).tolist(), flush=True)
    assert np.array_equal(branch, want["branch"])
    assert (np.abs(got["h"].cpu().numpy()[ps] - want["h"][ps]) <= 1e-9 * 2.4 * want["s"][ps]).all()
