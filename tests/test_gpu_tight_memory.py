"""Calls where device memory runs short: scratch that only makes a call faster
is given up when it does not fit beside what the call needs, and blocks kept
for later calls go back to the device first.  A test finds the least free
memory with which a call is carried out (by halving, to 8 MB) and compares it
with that of the same call by other means."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MB = 1 << 20


def free_bytes():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


class Hold:
    """Device memory taken past torch's allocator: all but n_bytes (to 4 MB)."""

    def __init__(self, n_bytes):
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.blocks = []
        while (more := free_bytes() - n_bytes) > 4 * MB:
            p = ctypes.c_void_p()
            assert self.hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(more - 2 * MB)) == 0
            self.blocks.append(p)

    def free(self):
        for p in self.blocks:
            self.hip.hipFree(p)
        self.blocks = []


@pytest.fixture(scope="module")
def pkg():
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pkg.Context(0).close()  # the runtime's own first allocations
    hold = Hold(4096 * MB)  # most of the device once: it takes a second
    yield pkg
    hold.free()


def least(pkg, call, most):
    """The least free memory (within 8 MB, at most `most`) with which call(n_bytes)
    succeeds; call leaves n_bytes free by itself."""
    lo, hi = 0, most
    while hi - lo > 8 * MB:
        mid = (lo + hi) // 2
        try:
            call(mid)
            hi = mid
        except pkg.SphmapError as e:
            assert e.code == -2, e  # SPHMAP_ENOMEM
            lo = mid
    print("   least free memory", hi >> 20, "MB", flush=True)
    return hi


def test_voronoi_without_room_for_kept_cells(pkg):
    n = 60000
    kept = n * 1232  # bytes of finished cells kept between the count and the arrays
    print("case: voronoi in tight memory", n, flush=True)
    g = torch.as_tensor(np.random.default_rng(2).random((n, 3)), device="cuda")
    ctx = pkg.Context(0)
    dt, _ = pkg.build_voronoi(ctx, g, n_lloyd=0)
    want = dt.export()
    dt.free()
    ctx.close()

    def call(cap, n_bytes):
        ctx = pkg.Context(0, workspace_bytes=cap)
        hold = Hold(n_bytes)
        try:
            dt, _ = pkg.build_voronoi(ctx, g, n_lloyd=0)
            hold.free()
            t = dt.export()
            dt.free()
        finally:
            hold.free()
            ctx.close()
        assert np.array_equal(want.vertices, t.vertices) and np.array_equal(want.face_vtx, t.face_vtx)

    # a context with a workspace cap keeps no cells
    bare = least(pkg, lambda b: call(8 << 30, b), 1600 * MB)
    assert least(pkg, lambda b: call(0, b), 1600 * MB) < bare + kept // 2


def test_blocks_of_a_grid_freed_under_a_cap(pkg):
    """A cap set after the grid was made: its blocks go to the device."""
    print("case: grid freed under a cap set later", flush=True)
    g = torch.as_tensor(np.random.default_rng(5).random((20000, 3)), device="cuda")
    ctx = pkg.Context(0)
    pkg.build_voronoi(ctx, g, n_lloyd=0)[0].free()
    ctx.set_pool_limit(0)
    ctx.set_pool_limit(8 << 30)
    base = free_bytes()
    dt, _ = pkg.build_voronoi(ctx, g, n_lloyd=0)
    ctx.set_pool_limit(0)  # what the build itself gave back
    ctx.set_pool_limit(8 << 30)
    assert base - free_bytes() > 100 * MB
    ctx.set_workspace_limit(8 << 30)
    dt.free()
    left = base - free_bytes()
    ctx.close()
    assert left < 8 * MB


def held_by_grid(pkg, ctx, build, base):
    """What the device lacks while a grid is there, its maker's pool emptied."""
    dt = build()
    ctx.set_pool_limit(0)
    got = base - free_bytes()
    ctx.set_pool_limit(8 << 30)
    return dt, got


def test_grids_stay_within_the_stated_footprint(pkg):
    """sphmap_estimate_footprint bounds what a grid holds, also when it is made
    from blocks that a larger grid gave back."""
    print("case: footprint of a grid from the pool", flush=True)
    rng = np.random.default_rng(3)
    big, small = (torch.as_tensor(rng.random((n, 3)), device="cuda") for n in (30000, 16500))
    ctx = pkg.Context(0)
    for g in (big, small):  # the scratch reaches its size
        pkg.build_voronoi(ctx, g, n_lloyd=0)[0].free()
    ctx.set_pool_limit(0)
    ctx.set_pool_limit(8 << 30)
    base = free_bytes()
    pkg.build_voronoi(ctx, big, n_lloyd=0)[0].free()
    dt, got = held_by_grid(pkg, ctx, lambda: pkg.build_voronoi(ctx, small, n_lloyd=0)[0], base)
    est = ctx.estimate_footprint(1, dt.export())["tessellation"]
    dt.free()
    ctx.close()
    print("   holds", got >> 20, "MB, stated bound", est >> 20, "MB", flush=True)
    assert got <= est


@pytest.mark.parametrize("what", ["neighbours", "plan"])
def test_pool_blocks_give_way(pkg, workloads, what):
    """A freed grid's blocks in the pool are the device's again for whatever the
    context allocates next."""
    print("case: pool gives way to", what, flush=True)
    n = 40000 if what == "neighbours" else 20000
    pos, m, h, _ = workloads.make_cloud("uniform", n, seed=6)
    tess = workloads.voronoi(pos)
    x, mm, hh = (torch.as_tensor(a, device="cuda") for a in (pos, m, h))
    ctx, hold = pkg.Context(0), None
    try:
        dt = ctx.upload(tess, neighbours=False)
        pkg.map_particles_to_cells(ctx, dt, x, hh, mm)  # scratch
        for d in [ctx.upload(tess) for _ in range(2)]:
            d.free()
        hold = Hold(4 * MB)
        if what == "neighbours":
            assert dt.set_face_neighbours(tess.face_nbr) > 0
        else:
            plan = pkg.BatchPlan(ctx, [dt], [x], [hh], [mm])
            plan.run()
            torch.cuda.synchronize()
            plan.free()
        hold.free()
        dt.free()
    finally:
        if hold:
            hold.free()
        ctx.close()


def test_binary64_mapping_without_room_for_records(pkg, workloads):
    """The binary64 edge kernel's face records (400 MB and more) are given up:
    the call needs what the one-lane kernel of a capped context needs."""
    print("case: binary64 mapping in tight memory", flush=True)
    pos, m, h, _ = workloads.make_cloud("uniform", 20000, seed=6)
    tess = workloads.voronoi(pos)
    x, mm, hh = (torch.as_tensor(a, device="cuda") for a in (pos, m, h))
    out = {k: torch.empty(tess.n_cells, dtype=torch.float64, device="cuda") for k in ("out_mass", "out_density")}
    mass = {}

    def call(cap, n_bytes):
        ctx, hold = pkg.Context(0, workspace_bytes=cap), None
        try:
            dt = ctx.upload(tess)
            hold = Hold(n_bytes)
            pkg.map_particles_to_cells(ctx, dt, x, hh, mm, precision="fp64", with_coverage=False, **out)
            torch.cuda.synchronize()
            mass[cap] = out["out_mass"].clone()
            hold.free()
            dt.free()
        finally:
            if hold:
                hold.free()
            ctx.close()

    bare = least(pkg, lambda b: call(64 << 30, b), 1200 * MB)
    assert least(pkg, lambda b: call(0, b), 1200 * MB) < bare + 100 * MB
    assert torch.allclose(mass[0], mass[64 << 30], rtol=1e-12, atol=0.0)


def test_pool_gives_way_to_a_grid_under_a_cap(pkg, workloads):
    """Blocks that lay in the pool before a cap was set are no use to a grid made
    under it, but their memory is."""
    print("case: pool gives way to a grid under a cap", flush=True)
    pos, m, h, _ = workloads.make_cloud("uniform", 10000, seed=6)
    tess = workloads.voronoi(pos)
    ctx, hold = pkg.Context(0), None
    try:
        first = ctx.upload(tess)
        for d in [ctx.upload(tess) for _ in range(2)]:
            d.free()
        ctx.set_workspace_limit(4 << 30)
        hold = Hold(4 * MB)
        dt = ctx.upload(tess)
        assert all(torch.equal(a, b) for a, b in zip(dt.cell_info(), first.cell_info()))
        hold.free()
        dt.free()
        first.free()
    finally:
        if hold:
            hold.free()
        ctx.close()
