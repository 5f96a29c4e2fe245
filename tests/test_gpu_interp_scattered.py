"""Interpolation onto few particles of a large set, far apart from each other:
wavefronts hold fewer particles then.  Every value is that of the whole cloud's
call, bit for bit, whatever the count (below and above the powers of two at
which the particles a wavefront change, at one batch of entries and above), and
64 scattered particles take little more time than the slowest of them alone
(several times as long with 64 to a wavefront; least of ten, a factor of two
allowed)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mixed(workloads):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pos = workloads.turbulent_cloud(300000, 3, grid=64)
    ctx = pkg.Context(0)
    x = torch.as_tensor(pos, device="cuda")
    h, m = (torch.full((len(pos),), v, dtype=torch.float64, device="cuda") for v in (0.02, 1.0 / len(pos)))
    ps = pkg.build_pseudo_particles(ctx, x, h, m, [[0.4, 0.5, 0.6]], r_part=0.2, theta=0.3)
    vals = torch.stack([torch.sin(7 * ps["xyz"][:, 0]), ps["xyz"][:, 1], torch.cos(5 * ps["xyz"][:, 2])], 1)
    full = pkg.interpolate_to_particles(ctx, x, ps, vals)
    yield pkg, ctx, x, ps, vals, full
    ctx.close()


def subset(ps, idx):
    return dict(ps, owner=ps["owner"][idx].contiguous())


@pytest.mark.parametrize("n", [1, 2, 63, 65, 4095, 4097, 8191, 8193, 16385, 131073, 262145])
def test_values_of_the_whole_cloud(mixed, n):
    pkg, ctx, x, ps, vals, full = mixed
    print("case: scattered", n, "of", len(x), "entries", ps["kind"].shape[0], flush=True)
    idx = torch.as_tensor(np.random.default_rng(n).choice(len(x), n, replace=False), device="cuda")
    for k in (1, 3):
        out = pkg.interpolate_to_particles(ctx, x[idx], subset(ps, idx), vals[:, :k].contiguous())
        assert torch.equal(out, full[idx, :k])


@pytest.mark.parametrize("ne", [1, 63, 64, 65, 129])
def test_few_entries(ne, oracle):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: few entries", ne, flush=True)
    g = np.random.default_rng(ne)
    n, epos, eh = 5003, g.random((ne, 3)), g.uniform(0.05, 0.4, ne)
    kind = (g.random(ne) < 0.8).astype(np.int32)
    pos, owner, val = g.random((n, 3)), g.integers(0, ne, n), g.uniform(-1, 1, (ne, 2))
    ctx = pkg.Context(0)
    dev = {k: torch.as_tensor(v, device="cuda") for k, v in dict(xyz=epos, h=eh, kind=kind, owner=owner).items()}
    out = pkg.interpolate_to_particles(ctx, pos, dev, val).cpu().numpy()
    ctx.close()
    assert np.abs(out - oracle.interpolate(pos, owner, epos, eh, kind, val)).max() <= 1e-12


def test_time_of_scattered_particles(mixed):
    pkg, ctx, x, ps, vals, full = mixed
    far = torch.nonzero(ps["kind"][ps["owner"]] == 1).flatten()
    idx = far[torch.linspace(0, len(far) - 1, 64, device="cuda").long()]

    def best(sel):
        xs, sub, t = x[sel].contiguous(), subset(ps, sel), []
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            pkg.interpolate_to_particles(ctx, xs, sub, vals)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)
    alone, together = max(best(idx[k:k + 1]) for k in range(64)), best(idx)
    print(f"case: time of scattered particles {1e6 * alone:.0f} {1e6 * together:.0f} us", flush=True)
    assert together < 2.0 * alone
