"""The benchmark's cost model of the interpolation by rings, on the CPU: its (column, ring) pairs and entries
against the schedules that the library's own plan builder makes for the operator's nodes, and the bytes and
operations built from them."""
import subprocess
from types import SimpleNamespace

import numpy as np
import pytest

import bench
from oracle import ddi_oracle as O
from test_ring_blocks import blocks  # noqa: F401

L = 8.0
PLANS = [((32, 32, 32), (32, 16, 32), 14), ((16, 32, 24), (9, 7, 13), 9), ((24, 16, 64), (11, 6, 18), 5)]


@pytest.mark.parametrize("n,quad,w", PLANS)
def test_ring_model_counts_the_schedules_pairs_and_entries(blocks, n, quad, w):  # noqa: F811
    r = subprocess.run([blocks, *map(str, n), *map(str, quad), f"{0.9 * 10.0 ** -(w - 2):g}", "0", "1"], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    entries, pairs = [int(v) for v in r.stdout.splitlines()[1].split()[6:8]]
    prob = O.DDIProblem(dim=3, n=n, L=(L,) * 3, dip_n=(0.0, 0.0, 1.0), n_rad=quad[0], n_pol=quad[1], n_azi=quad[2])
    nodes, c = O.ddi_nodes(prob)
    kept = int(np.sum(bench.kept_nodes(nodes.index, quad)))
    window = 2 * n[2]
    plan = SimpleNamespace(dim=3, shape=n, L=(L,) * 3, nodes=lambda: (nodes.index, nodes.k, c),
                           info={"n_fine": tuple(2 * v for v in n), "width": w, "m_half": kept, "apply_window": window,
                                 "spread_entries": 0})
    assert bench.ring_counts(plan, quad) == (pairs, entries)
    b, f = bench.stage_model(plan, 8, 16, quad)["interp"]
    assert f == 4.0 * 64 * w * pairs + 4.0 * w * w * kept
    assert b == 4 * n[0] * n[1] * window * 16 + kept * (256 + 8 + 16) + 16 * pairs + 12 * entries
