"""The blocks of the FP64 3D interpolation by rings.

CPU: no block of these plans holds more than 128 entries (its rounds run one after the other), also where one
ring has more than that over a column (rules with many azimuthal nodes); where the entries make thousands of
blocks the limit rises to entries / 4096, at most 1024.  No block reaches beyond the
last-axis window, whose neighbourhood the transforms never write, and the blocks hold every (column, node)
pair of the tile lists once at the right offsets, also for nodes beyond the Nyquist box."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1504_02897_amd", "csrc")
BLOCK_ENTRIES = 128
# n, quad, tol, split, nyquist_mask, whether a ring has more entries over a column than a block takes
PLANS = [((16, 16, 16), (5, 5, 400), 1e-13, 0, 1, True), ((32, 32, 32), (4, 4, 4096), 1e-7, 0, 1, True),
         ((16, 32, 24), (3, 4, 301), 1e-9, 0, 1, True), ((32, 32, 32), (9, 6, 257), 1e-15, 0, 0, True),
         ((64, 64, 64), (16, 13, 32), 1e-13, 1, 1, False), ((48, 16, 64), (31, 15, 34), 1e-11, 0, 1, False),
         ((128, 128, 128), (1, 2, 128), 1e-15, 0, 1, False), ((32, 32, 32), (40, 20, 400), 1e-13, 0, 1, True)]


def build_driver(tmp_path_factory, name):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the ROCm headers are not available")
    exe = str(tmp_path_factory.mktemp("rings") / name)
    cmd = [gxx, "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           os.path.join(ROOT, "tests", "host", name + ".cpp"), os.path.join(CSRC, "plan.cpp"),
           os.path.join(CSRC, "rings.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    return build_driver(tmp_path_factory, "ring_blocks")


@pytest.mark.parametrize("n,quad,tol,split,mask,full", PLANS)
def test_no_block_is_longer_than_its_limit(blocks, n, quad, tol, split, mask, full):
    r = subprocess.run([blocks, *map(str, n), *map(str, quad), str(tol), str(split), str(mask)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    lines = [[int(v) for v in ln.split()] for ln in r.stdout.splitlines()]
    assert len(lines) == 2
    for _, count, longest, over, outside, faults, entries, _ in lines:
        assert count > 0 and outside == 0 and faults == 0
        assert longest <= min(max(entries // 4096, BLOCK_ENTRIES), 1024)
        assert (over > 0) == full



def test_rings_of_the_largest_rule_need_memory_for_its_nodes_only(tmp_path_factory):
    """65536 x 65536 radial and polar nodes, four of them inside the box: 1 GiB of address space is plenty."""
    exe = build_driver(tmp_path_factory, "ring_index")
    r = subprocess.run(["bash", "-c", f"ulimit -v 1048576 && exec {exe}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    rings = [int(v) for v in r.stdout.split()]
    # rings in the rule's order: (0, 65535) holds nodes 1 and 3, then (65535, 0) and (65535, 65535)
    assert rings == [3, 2, 0, 1, 0]


# ------------------------------------------------------------------ on the GPU
def kernel_model(n, L, w, k):
    """The NUFFT's own model in 64 bits: per axis the deconvolution factors D and each node's kernel weights
    over the fine axis (exponential-of-semicircle kernel, shape 2.30 w, twice oversampled)."""
    beta = 2.30 * w

    def psi(z):
        s = 1.0 - (2.0 * z / w) ** 2
        return np.where(s > 0.0, np.exp(beta * (np.sqrt(np.maximum(s, 0.0)) - 1.0)), 0.0)

    gx, gw = np.polynomial.legendre.leggauss(128)
    z = 0.25 * w * (gx + 1.0)
    D, W, S = [], [], []
    for a in range(3):
        nf = 2 * n[a]
        m = np.arange(n[a]) - n[a] // 2
        D.append(1.0 / (0.5 * w * np.sum(gw * psi(z) * np.cos(2.0 * np.pi * m[:, None] * z / nf), axis=1)))
        tau = k[:, a] * (2.0 * L[a] / n[a]) * nf / (2.0 * np.pi)
        l0 = np.ceil(tau - 0.5 * w).astype(np.int64)
        rows = np.zeros((k.shape[0], nf))
        for i in range(w):
            rows[np.arange(k.shape[0]), (l0 + i) % nf] += psi(l0 + i - tau)
        W.append(rows)
        S.append(float(0.5 * w * np.sum(gw * psi(z))))
    return D, W, S


def fine_modes(n):
    """Fine-grid place of each compact index (mode 0 at the box centre)."""
    return [(np.arange(v) - v // 2) % (2 * v) for v in n]


def model_type2(rho, cell, D, W):
    n = rho.shape
    pad = np.zeros([2 * v for v in n], dtype=np.complex128)
    pad[np.ix_(*fine_modes(n))] = rho * D[0][:, None, None] * D[1][None, :, None] * D[2]
    F = np.fft.fftn(pad)
    out = np.empty(W[0].shape[0], dtype=np.complex128)
    for s in range(0, out.size, 256):
        e = slice(s, s + 256)
        t = F @ W[2][e].T                                    # [x, y, q]
        out[e] = np.sum(W[0][e].T * np.sum(t * W[1][e].T[None], axis=1), axis=0)
    return cell * out


def model_type1(g, D, W):
    n = [d.size for d in D]
    F = np.zeros([2 * v for v in n], dtype=np.complex128)
    for s in range(0, g.size, 256):
        e = slice(s, s + 256)
        t = (g[e, None] * W[0][e])[:, :, None] * W[1][e][:, None, :]             # [q, x, y]
        F += np.tensordot(t, W[2][e], axes=(0, 0))
    F = np.fft.ifftn(F) * F.size
    return F[np.ix_(*fine_modes(n))].real * (D[0][:, None, None] * D[1][None, :, None] * D[2])


def half_factors(index, quad):
    """2 for the member of a +-k pair that the operator keeps (the first in the rule's order), 0 for the other, 1
    without a partner.  Not all ones: a node on an axis and its partner differ by the kernel's edge value."""
    nrad, npol, nazi = quad
    if nazi % 2:
        return np.ones(len(index))
    a, b, c = index.T.astype(np.int64)
    mine = (a * npol + b) * nazi + c
    other = (a * npol + npol - 1 - b) * nazi + (c + nazi // 2) % nazi
    return np.where(np.isin(other, mine), np.where(mine < other, 2.0, 0.0), 1.0)


GPU_PLANS = [((16, 16, 16), (5, 5, 400), 14, True), ((16, 32, 24), (3, 4, 301), 9, True), ((32, 32, 32), (9, 6, 257), 16, False),
             ((8, 16, 8), (6, 5, 260), 4, True), ((32, 16, 48), (13, 7, 30), 16, True)]


@pytest.mark.gpu
@pytest.mark.parametrize("n,quad,w,mask", GPU_PLANS)
def test_interpolation_matches_its_model_to_rounding(n, quad, w, mask):
    """type-2 over every node and the operator (half of the nodes), against the NUFFT's own model in numpy: the
    kernel's aliasing error is on both sides, so what is left is rounding."""
    import torch

    from paper_1504_02897_amd.ddi import DDIPlan

    L = (8.0, 6.0, 5.0)
    plan = DDIPlan(3, n, L, dip_n=(0.6, 0.0, 0.8), quad=quad, kernel_width=w, nyquist_mask=mask)
    index, k, c = plan.nodes()
    D, W, S = kernel_model(n, L, w, k)
    rng = np.random.default_rng(5)
    g = [np.exp(-(np.arange(v) - v / 2 + 0.3) ** 2 / (0.12 * v) ** 2) for v in n]
    rho = g[0][:, None, None] * g[1][None, :, None] * g[2] * (1.0 + 0.3 * rng.standard_normal(n))
    # rounding of the exponentials (arguments up to beta), of three transforms and of the sums; a
    # deconvolution factor is good to eps phihat(0) D (a sum with terms up to 1)
    eps = 2.0 ** -52
    ops = 3.0 * (2.30 * w + 8.0) + 9.0 * np.log2(2 * max(n)) + 3.0 * w
    grow = 1.0 + 8.0 / ops * sum(S[a] * D[a].reshape([-1 if i == a else 1 for i in range(3)]) for a in range(3))
    amp = D[0][:, None, None] * D[1][None, :, None] * D[2] * grow
    rows = [float(np.max(np.sum(W[a], axis=1))) for a in range(3)]
    scale = plan.cell * np.sum(np.abs(rho) * amp) * rows[0] * rows[1] * rows[2]
    x = torch.from_numpy(rho).cuda()
    got = plan.type2(x).cpu().numpy()
    want = model_type2(rho, plan.cell, D, W)
    assert np.max(np.abs(got - want)) <= ops * eps * scale
    phi = plan.apply(x).cpu().numpy()
    ref = model_type1(half_factors(index, quad) * c * want, D, W)
    # per point: the node values' own error and the way back, each bounded as above
    bound = 2.0 * ops * eps * scale * np.sum(np.abs(c)) * rows[0] * rows[1] * rows[2] * amp
    assert np.all(np.abs(phi - ref) <= bound)
