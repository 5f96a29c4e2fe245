"""What a batch plan's graph writes to is the plan's own: a plan of a context
that has mapped nothing else, and one whose context afterwards grows its
scratch, gives it back under a cap and takes new blocks for other work, replay
the single calls' results bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def clouds(workloads, sizes):
    out = []
    for n in sizes:
        pos, m, h, _ = workloads.make_cloud("uniform", n, seed=n)
        out.append((workloads.voronoi(pos), *(torch.as_tensor(a, device="cuda") for a in (pos, h, m))))
    return out


def same(plan, want):
    counts, over = plan.check()
    assert not over
    for k, r in enumerate(want):
        assert torch.equal(plan.mass[k], r.mass) and torch.equal(plan.coverage[k], r.coverage), k


def test_plan_of_a_fresh_context(workloads):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: plan of a fresh context", flush=True)
    c = clouds(workloads, (700, 1500))
    ref = pkg.Context(0)
    want = [pkg.map_particles_to_cells(ref, ref.upload(t), x, h, m) for t, x, h, m in c]
    ctx = pkg.Context(0)
    plan = pkg.BatchPlan(ctx, [ctx.upload(t) for t, _, _, _ in c], *([a[k] for a in c] for k in (1, 2, 3)))
    for _ in range(3):
        plan.run()
        same(plan, want)
    plan.free()
    ctx.close()
    ref.close()


def test_plan_beside_changing_scratch(workloads):
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: plan beside changing scratch", flush=True)
    c = clouds(workloads, (700, 1500))
    (t, x, h, m), = clouds(workloads, (20000,))
    ctx = pkg.Context(0)
    grids = [ctx.upload(a[0]) for a in c]
    want = [pkg.map_particles_to_cells(ctx, d, *a[1:]) for d, a in zip(grids, c)]
    plan = pkg.BatchPlan(ctx, grids, *([a[k] for a in c] for k in (1, 2, 3)))
    plan.run()
    same(plan, want)
    big = ctx.upload(t)
    ref = pkg.map_particles_to_cells(ctx, big, x, h, m)  # the scratch grows past the plan's
    plan.run()
    same(plan, want)
    ctx.set_workspace_limit(1 << 20)  # and is given back
    ctx.set_workspace_limit(0)
    blocks = [torch.full((64 << 20,), 255, dtype=torch.uint8, device="cuda") for _ in range(16)]
    for _ in range(3):
        plan.run()
        same(plan, want)
        assert torch.equal(pkg.map_particles_to_cells(ctx, big, x, h, m).mass, ref.mass)
    assert all(bool((b == 255).all()) for b in blocks)
    assert ctx.sync_status() == 0
    c[0][3][0] = float("nan")  # the status word is still the one that the plan knows
    plan.run()
    assert ctx.sync_status() & pkg.STATUS_NONFINITE_MASS
    plan.free()
    ctx.close()
