"""The FP64 3D interpolation by rings.

CPU: the ring schedules against the tile lists of the same plan (every (column, node) pair once, every
index consistent, a node's weights over its entries adding up to its whole kernel), over shapes with
and without a gap in the last-axis window, odd quadrature sizes, one node, a small ball.
GPU: type-2 at every node against direct sums in 64 bits, on grids whose blocks wrap round the last
axis, end at the window's edge, or hold one ring of one node."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1504_02897_amd", "csrc")
SHAPES = [((32, 32, 32), (32, 16, 32), 1e-13, 0), ((8, 8, 8), (10, 5, 11), 1e-7, 0), ((24, 12, 8), (9, 7, 13), 1e-5, 0),
          ((16, 24, 12), (9, 7, 13), 1e-10, 0), ((64, 16, 32), (31, 15, 34), 1e-13, 0), ((8, 8, 8), (1, 1, 1), 1e-5, 0),
          ((64, 64, 64), (16, 13, 32), 1e-13, 1)]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the ROCm headers are not available")
    exe = str(tmp_path_factory.mktemp("rings") / "ring_tables")
    cmd = [gxx, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           os.path.join(ROOT, "tests", "host", "ring_tables.cpp"), os.path.join(CSRC, "plan.cpp"),
           os.path.join(CSRC, "rings.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("n,quad,tol,split", SHAPES)
def test_ring_schedules_match_the_tile_lists(driver, n, quad, tol, split):
    r = subprocess.run([driver, *map(str, n), *map(str, quad), str(tol), str(split)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    lines = [ln.split() for ln in r.stdout.splitlines()]
    assert len(lines) == 2
    for _, entries, faults, err in lines:
        assert int(entries) > 0 and int(faults) == 0
        assert float(err) <= 48 * 2.3e-16 * 4          # sums of at most 48 weights, regrouped


@pytest.mark.gpu
@pytest.mark.parametrize("n,quad,tol,split", SHAPES)
def test_ring_interpolation_matches_direct_sums(n, quad, tol, split):
    import torch

    from paper_1504_02897_amd.ddi import DDIPlan

    plan = DDIPlan(3, n, (8.0,) * 3, dip_n=(0.6, 0.0, 0.8), quad=quad, tol=tol, split=bool(split))
    rng = np.random.default_rng(3)
    x = [-8.0 + 16.0 / v * np.arange(v) for v in n]
    g = [np.exp(-(a / 3.0) ** 2) for a in x]
    rho = g[0][:, None, None] * g[1][None, :, None] * g[2] * (1.0 + 0.3 * rng.standard_normal(n))
    got = plan.type2(torch.from_numpy(rho).cuda()).cpu().numpy()
    _, k, _ = plan.nodes()
    ph = [np.exp(-1j * np.outer(k[:, a], x[a])) for a in range(3)]
    want = np.einsum("qx,qxz,qz->q", ph[0], np.einsum("qy,xyz->qxz", ph[1], rho, optimize=True), ph[2],
                     optimize=True) * plan.cell
    # the NUFFT's aliasing error is bounded by a few tol of sum |rho| per axis
    assert np.max(np.abs(got - want)) <= 30.0 * tol * plan.cell * np.sum(np.abs(rho))
