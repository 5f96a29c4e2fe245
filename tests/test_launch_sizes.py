"""Launches that step through their items: their sizes stay below what one
launch may have for every count the header admits (checked on the CPU), and
the items past the first step are done (GPU)."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_15227_amd", "csrc")


def run_host(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include "common.hpp"\nusing namespace sphmap;\nint main() {\n' + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-w", str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


def test_octant_launches_below_the_limit(tmp_path):
    # eight lanes a node, levels bounded by n < 2^31
    out = run_host(tmp_path, "for (int64_t n : {1ll, 31ll, 32ll, 33ll, 1ll << 20, 1ll << 29, (1ll << 31) - 1})"
                             ' printf("%u ", strided_blocks(8 * n));')
    blocks = [int(v) for v in out.split()]
    assert blocks[:4] == [1, 1, 1, 2]
    assert max(blocks) * 256 < 2 ** 32 and min(blocks) > 0


@pytest.mark.gpu
def test_octree_levels_of_several_steps(oracle):
    torch = pytest.importorskip("torch")
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case: octree levels of more nodes than a launch holds", flush=True)
    n = 300011  # levels of up to 200,000 nodes; a launch holds 131,072
    x = np.random.default_rng(8).random((n, 3))
    m, h, src = np.full(n, 1.0 / n), np.full(n, 0.02), [[0.5, 0.5, 0.5]]
    kw = dict(r_part=3.0, theta=0.5, leaf_max=1)
    ref = oracle.pseudo_build(x, m, h, src, **kw)
    ctx = pkg.Context(0)
    got = pkg.build_pseudo_particles(ctx, x, h, m, src, **kw)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in got.items() if k != "stats"}
    ctx.close()
    assert got["stats"]["n_nodes"] == ref["n_nodes"] > 131072
    assert np.array_equal(g["first"], ref["first"]) and np.array_equal(g["owner"], ref["owner"])
    assert np.array_equal(g["label"].view(np.uint64), ref["label"])


@pytest.mark.gpu
def test_grid_preparation_of_several_launches(oracle):
    torch = pytest.importorskip("torch")
    import paper_2410_15227_amd as pkg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 530003  # a launch prepares 524,288 cells
    print("case: grid of", n, "cells", flush=True)
    g = np.random.default_rng(9).random((n, 3))
    ctx = pkg.Context(0)
    dt, _ = pkg.build_voronoi(ctx, g, n_lloyd=0)
    vol, rad = (a.cpu().numpy() for a in dt.cell_info())
    dt.free()
    ctx.close()
    cells = np.array([0, 7, 524287, 524288, 524289, n - 1])
    want, _ = oracle.voronoi_cells(g, cells)
    assert np.max(np.abs(vol[cells] - want) / want) < 1e-11
    assert abs(vol.sum() - 1.0) < 1e-11 and (rad > 0).all()
