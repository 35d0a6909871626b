"""What a user of the library has it do, as cases that can be timed and checked.

``listed()`` holds the fixed cases, ``draw(rng)`` more of the same ranges; ``prepare`` makes the
plan and the inputs on the GPU, ``run`` is one pass through the public entry points, ``work`` the
bytes and operations that pass cannot do without, and ``exact`` its outputs in 64 bits by direct
sums over the quadrature (no NUFFT and none of this package's code).

A case is a dict of plain values:
  op      apply   Phi = A rho
          grad    Phi = A rho and the gradient of <Phi, g> by autograd (forward and backward)
          filter  type-2, multiplication by the caller's own factors per node, type-1
          energy  GPE energies and gradient
          flow    one gradient-flow step (n_inner Fourier iterations)
          dynamics  new dipole axis, then one time-splitting step
  dim, n0..n2, L0..L2   grid (2D uses axes 0 and 1)
  n_rad, n_pol, n_azi, tol, prec, split, stretch   the plan's quadrature, accuracy and form
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1504_02897_amd.ddi import DDIPlan, ddi_apply


def _case(name, op, n, L, quad, tol=1e-13, prec="fp64", split=False, stretch=1.0, n_inner=1):
    dim = len(n)
    case = {"op": op, "dim": dim}
    for i in range(dim):
        case[f"n{i}"] = int(n[i])
        case[f"L{i}"] = float(L[i])
    case.update(n_rad=int(quad[0]), n_pol=int(quad[1]), n_azi=int(quad[2]), tol=float(tol), prec=prec,
                split=bool(split), stretch=float(stretch), n_inner=int(n_inner))
    if name is not None:
        case = {"name": name, **case}
    return case


def listed():
    return [
        # the package's small 3D problem (c1_32): one Phi of a compact density, where launches count
        _case("apply_32", "apply", (32,) * 3, (8.0,) * 3, (32, 16, 32)),
        # the headline evaluation (c2_128): Phi of a mixture at 128^3 in FP64
        _case("apply_128", "apply", (128,) * 3, (12.0,) * 3, (96, 48, 96)),
        # training through the operator at the paper's 96^3 (Table 7's grid): Phi and its gradient
        _case("grad_96", "grad", (96,) * 3, (12.0,) * 3, (72, 36, 72)),
        # the headline evaluation in mixed precision
        _case("apply_128_mixed", "apply", (128,) * 3, (12.0,) * 3, (96, 48, 96), tol=1e-7, prec="mixed"),
        # the large evaluation (c4_256): Phi at 256^3 in mixed precision
        _case("apply_256_mixed", "apply", (256,) * 3, (16.0,) * 3, (128, 64, 128), tol=1e-7, prec="mixed"),
        # the quasi-2D evaluation (c3_512)
        _case("apply_2d_512", "apply", (512, 512), (16.0, 16.0), (128, 1, 256)),
        # training through the quasi-2D operator on a smaller, non-square grid in mixed precision
        _case("grad_2d_192_mixed", "grad", (192, 256), (12.0, 16.0), (93, 1, 186), tol=1e-6, prec="mixed"),
        # the split evaluation (Eq. 3.9) of the headline density
        _case("apply_128_split", "apply", (128,) * 3, (12.0,) * 3, (32, 32, 64), split=True),
        # a user's own interaction through the two NUFFT halves, non-cubic grid, odd quadrature sizes
        _case("filter_64", "filter", (64, 96, 48), (8.0, 12.0, 6.0), (45, 23, 46), tol=1e-10),
        # energies and gradient of a state at 128^3 (the optimiser's call), harmonic trap
        _case("energy_128", "energy", (128,) * 3, (8.0,) * 3, (96, 48, 96)),
        # a step of the ground-state flow with a converged inner solve (Table 7: 30 iterations)
        _case("flow_96", "flow", (96,) * 3, (12.0,) * 3, (72, 36, 72), n_inner=30),
        # a step of the rotating-dipole dynamics (c8_dip_rot): new axis, time-splitting step, split plan
        _case("dynamics_128_split", "dynamics", (128,) * 3, (8.0,) * 3, (32, 32, 64), split=True),
    ]


_SIZES = (16, 24, 32, 48, 64, 96, 128, 192, 256)


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _grid_size(rng, lo, hi):
    """A grid size of the library (2^a or 3 * 2^a) in [lo, hi], uniform in its logarithm."""
    v = _log_uniform(rng, lo, hi)
    return min((s for s in _SIZES + (384, 512) if lo <= s <= hi), key=lambda s: abs(math.log(s / v)))


def draw(rng):
    """One more case: any operation, 2D or 3D, both precisions, whole ball or split, other box shapes."""
    op = rng.choice(("apply", "apply", "grad", "filter", "energy", "flow", "dynamics"))
    dim = 2 if rng.random() < 0.25 else 3
    prec = rng.choice(("fp64", "mixed"))
    split = op != "filter" and rng.random() < 0.25
    if dim == 3:
        top = 256 if prec == "mixed" and op == "apply" else 128     # cost: at most that of the 256^3 case
        base = _grid_size(rng, 24, top)
        n = [base] * 3
        if rng.random() < 0.5:                                        # one axis shorter or longer
            n[rng.randrange(3)] = _grid_size(rng, max(24, base // 2), min(128, 2 * base))
    else:
        n = [_grid_size(rng, 96, 512), _grid_size(rng, 64, 512)]
    h = rng.uniform(0.12, 0.3) if dim == 3 else rng.uniform(0.06, 0.2)
    L = [0.5 * h * v * rng.uniform(0.9, 1.1) for v in n]
    tol = 10.0 ** -rng.uniform(5.0, 7.5) if prec == "mixed" else 10.0 ** -rng.uniform(8.0, 13.5)
    if split:
        n_rad = rng.randint(12, 40)
        quad = (n_rad, rng.randint(12, 36) if dim == 3 else 1, 2 * rng.randint(12, 36))
        L = [min(L)] * dim                                            # the split's s follows the shortest side
    else:
        n_rad = min(128 if dim == 3 else 160, max(10, int(max(n) * rng.uniform(0.45, 0.9))))
        n_azi = 2 * max(5, int(n_rad * rng.uniform(0.4, 0.6 if dim == 3 else 1.0)))
        quad = (n_rad, max(4, int(n_rad * rng.uniform(0.4, 0.55))) if dim == 3 else 1, n_azi)
    stretch = rng.uniform(1.0, 2.0) if dim == 3 and not split and rng.random() < 0.2 else 1.0
    n_inner = rng.choice((1, 5, 30) if math.prod(n) <= 96 ** 3 else (1, 5)) if op == "flow" else 1
    return _case(None, op, n, L, quad, tol=tol, prec=prec, split=split, stretch=stretch, n_inner=n_inner)


# --------------------------------------------------------------------------------- inputs
_BETA, _LAM, _DT_FLOW, _DT_DYN = 103.58, 82.864, 0.02, 0.005


def _shape(case):
    return tuple(case[f"n{i}"] for i in range(case["dim"]))


def _box(case):
    return tuple(case[f"L{i}"] for i in range(case["dim"]))


def _axes(case):
    """x_l = -L + l h per axis, on the GPU."""
    return [torch.arange(n, dtype=torch.float64, device="cuda") * (2.0 * L / n) - L
            for n, L in zip(_shape(case), _box(case))]


def _along(v, axis, dim):
    return v.reshape([-1 if i == axis else 1 for i in range(dim)])


def _inputs(case, seed):
    """The density's wave function (a normalised mixture of Gaussian lumps with constant phases; in 2D
    with 10% random-phase noise, as the package's workloads), the dipole axes, a smooth cotangent and
    the plan's grid type."""
    dim, shape, L = case["dim"], _shape(case), _box(case)
    rng = np.random.default_rng(seed)
    ax = _axes(case)

    def lumps(count):
        out = torch.zeros(shape, dtype=torch.complex128, device="cuda")
        for _ in range(count):
            th = rng.uniform(0.0, 2.0 * math.pi)
            f = complex(math.cos(th), math.sin(th))
            for i in range(dim):
                c, w = rng.uniform(-0.25, 0.25) * L[i], rng.uniform(0.06, 0.2) * L[i]
                f = f * _along(torch.exp(-((ax[i] - c) ** 2) / (2.0 * w * w)), i, dim)
            out += f
        return out

    psi = lumps(int(rng.integers(1, 5 if dim == 3 else 7)))
    if dim == 2:
        xi = torch.from_numpy(rng.uniform(0.0, 1.0, size=shape)).cuda()
        eta = torch.from_numpy(rng.uniform(0.0, 2.0 * math.pi, size=shape)).cuda()
        psi = psi + 0.1 * psi.abs().max() * torch.polar(xi, eta)
    cell = math.prod(2.0 * Li / ni for ni, Li in zip(shape, L))
    psi = psi / torch.sqrt(cell * (psi.real ** 2 + psi.imag ** 2).sum())
    if dim == 3:
        axis = rng.standard_normal(3)
        axis = axis / np.linalg.norm(axis)
    else:
        t = rng.uniform(0.0, 2.0 * math.pi)
        axis = np.array([math.sin(math.pi / 4) * math.cos(t), math.sin(math.pi / 4) * math.sin(t), math.cos(math.pi / 4)])
    t2 = rng.uniform(0.0, 0.4)
    axis2 = np.array([math.sin(t2), 0.0, math.cos(t2)])
    g = lumps(2).real.contiguous()
    cdt = torch.complex64 if case["prec"] == "mixed" else torch.complex128
    rdt = torch.float32 if case["prec"] == "mixed" else torch.float64
    psi = psi.to(cdt)
    rho = (psi.real.double() ** 2 + psi.imag.double() ** 2).to(rdt)
    return {"psi": psi, "rho": rho, "g": g.to(rdt), "axis": tuple(axis), "axis2": tuple(axis2)}


def _gamma(case):
    return tuple((1.0, 1.0, 2.0)[: case["dim"]])


def _yukawa(kk):
    """The caller's own factors of the filter case: a screened Coulomb interaction 1 / (1 + |k|^2)."""
    return 1.0 / (1.0 + kk)


def prepare(case, seed):
    inp = _inputs(case, seed)
    dim = case["dim"]
    stretch = (1.0, 1.0, case["stretch"]) if dim == 3 else (1.0, 1.0, 1.0)
    plan = DDIPlan(dim, _shape(case), _box(case), dip_n=inp["axis"], quad=(case["n_rad"], case["n_pol"], case["n_azi"]),
                   tol=case["tol"], prec=case["prec"], split=case["split"], stretch=stretch)
    st = {"case": case, "plan": plan}
    op = case["op"]
    if op == "apply":
        st.update(rho=inp["rho"], out=torch.empty_like(inp["rho"]))
    elif op == "grad":
        st.update(rho=inp["rho"].requires_grad_(True), g=inp["g"])
    elif op == "filter":
        _, k, _ = plan.nodes()
        f = _yukawa(np.sum(k * k, axis=1)) * 1e-3
        st.update(rho=inp["rho"], f=torch.from_numpy(f).cuda().to(plan.real_dtype))
    else:
        st.update(psi=inp["psi"], axis2=inp["axis2"], out=torch.empty_like(inp["psi"]))
    return st


def run(state):
    plan, case = state["plan"], state["case"]
    op = case["op"]
    if op == "apply":
        return plan.apply(state["rho"], out=state["out"])
    if op == "grad":
        phi = ddi_apply(state["rho"], plan)
        (bar,) = torch.autograd.grad(phi, state["rho"], grad_outputs=state["g"])
        return phi.detach(), bar
    if op == "filter":
        return plan.type1(plan.type2(state["rho"]) * state["f"])
    if op == "energy":
        return plan.energy_grad(state["psi"], _BETA, _LAM, _gamma(case))
    if op == "flow":
        return plan.gf_step(state["psi"], _BETA, _LAM, _gamma(case), dt=_DT_FLOW, n_inner=case["n_inner"], out=state["out"])
    plan.set_dipole(state["axis2"])
    return plan.ts_step(state["psi"], _BETA, _LAM, _gamma(case), dt=_DT_DYN, out=state["out"])


# --------------------------------------------------------------------------------- quadrature (64 bits)
def _split_parameters(case):
    lt = math.log(1.0 / case["tol"])
    s = math.sqrt(lt) / min(_box(case))
    return s, s * math.sqrt(lt)


def _rings(case, axis):
    """The quadrature by radial shells: per radial node r, the polar nodes' (k_z, sin theta) and the
    azimuths' (cos, sin) with weights; the mask |k_i| <= pi / h_i and c = W Uhat / (2 pi)^d (times q for a
    split plan)."""
    dim, shape, L = case["dim"], _shape(case), _box(case)
    h = [2.0 * Li / ni for ni, Li in zip(shape, L)]
    S = np.array([1.0, 1.0, case["stretch"]])[:dim] if dim == 3 else np.ones(2)
    if case["split"]:
        s, kmax = _split_parameters(case)
    else:
        s, kmax = 0.0, math.pi * math.sqrt(sum(1.0 / (hi * Si) ** 2 for hi, Si in zip(h, S)))
    t, w = np.polynomial.legendre.leggauss(case["n_rad"])
    r, wr = 0.5 * kmax * (1.0 + t), 0.5 * kmax * w
    phi = 2.0 * math.pi * np.arange(case["n_azi"]) / case["n_azi"]
    wphi = 2.0 * math.pi / case["n_azi"]
    u, wu = np.polynomial.legendre.leggauss(case["n_pol"]) if dim == 3 else (np.zeros(1), np.ones(1))
    n = np.asarray(axis)
    R, U, P = np.meshgrid(r, u, phi, indexing="ij")
    su = np.sqrt(1.0 - U * U)
    k = [R * su * np.cos(P), R * su * np.sin(P)] + ([R * U] if dim == 3 else [])
    k = [ki * Si for ki, Si in zip(k, S)]
    W = wr[:, None, None] * R ** (dim - 1) * wu[None, :, None] * wphi * float(np.prod(S))
    kk = sum(ki * ki for ki in k)
    kn = sum(ki * ni for ki, ni in zip(k, n))
    if dim == 3:
        sym = 3.0 * kn * kn / kk - float(n @ n)
    else:
        sym = 3.0 * (kn * kn - n[2] * n[2] * kk) / (2.0 * np.sqrt(kk))
    q = 1.0
    if case["split"]:
        q = np.exp(-kk / (s * s)) if dim == 3 else torch.special.erfc(torch.from_numpy(np.sqrt(kk) / s)).numpy()
    inside = np.ones_like(kk, dtype=bool)
    for ki, hi in zip(k, h):
        inside &= np.abs(ki) <= math.pi / hi
    return k, kk, inside, W * inside / (2.0 * math.pi) ** dim * q, sym


def work(case):
    """Bytes and operations of one pass: the grids in and out, the fine-grid transforms and the kernel
    sums of the quadrature (w^d products per node of a +-k pair), whatever way they are done."""
    dim, shape = case["dim"], _shape(case)
    N = math.prod(shape)
    real = 4 if case["prec"] == "mixed" else 8
    _, _, inside, _, _ = _rings(case, (0.0, 0.0, 1.0))
    M = int(inside.sum())
    w = min(16, max(4, math.ceil(-math.log10(case["tol"])) + 1))
    op = case["op"]
    nfine = N * 2 ** dim
    fft = 5.0 * nfine * math.log2(nfine) / 2              # half the spectrum of a real field
    one = 2 * fft + 2 * 4.0 * (M if op == "filter" else M / 2) * w ** dim     # one Phi
    if case["split"]:
        one += 2 * fft
    full = 5.0 * N * math.log2(N)                           # one transform of the state
    applies = {"apply": 1, "grad": 2, "filter": 1, "energy": 2, "flow": 1, "dynamics": 1}[op]
    flops = applies * one
    nbytes = 2 * N * real                                   # one grid in, one out
    if op == "grad":
        nbytes = 4 * N * real
    elif op == "filter":
        nbytes += M * real
    elif op in ("energy", "flow", "dynamics"):
        nbytes = 4 * N * real
        flops += full * {"energy": 2, "flow": 1 + 2 * case["n_inner"], "dynamics": 4}[op]
    return {"bytes": float(nbytes), "flops": float(flops)}


# --------------------------------------------------------------------------------- exact outputs
def _direct(case, axis, rho, factors=None):
    """sum_q c_q Re[rhohat_q exp(i k_q . x)] by direct sums on the GPU in 64 bits, shell by shell: the
    sums over the last axis are shared by the azimuths of a ring.  factors (of |k|^2) replaces c_q."""
    dim = case["dim"]
    k, kk, inside, c, sym = _rings(case, axis)
    c = inside * factors(kk) if factors is not None else c * sym
    cell = math.prod(2.0 * L / n for n, L in zip(_shape(case), _box(case)))
    x = _axes(case)
    rho = rho.double()
    out = torch.zeros_like(rho)

    def phases(kv, xv):                                     # exp(i k x): [..., len(k), len(x)]
        a = kv.unsqueeze(-1) * xv
        return torch.complex(torch.cos(a), torch.sin(a))

    dev = [torch.from_numpy(np.ascontiguousarray(ki)).cuda() for ki in k]
    cd = torch.from_numpy(np.ascontiguousarray(c)).cuda()
    if dim == 2:
        ex = phases(dev[0].reshape(-1), x[0])
        ey = phases(dev[1].reshape(-1), x[1])
        cf = cd.reshape(-1)
        for s in range(0, cf.numel(), 8192):
            a, b = ex[s:s + 8192], ey[s:s + 8192]
            t = (a.conj() @ rho.to(torch.complex128)) * b.conj()
            g = cf[s:s + 8192] * cell * t.sum(1)
            out += ((g.unsqueeze(1) * a).transpose(0, 1).contiguous() @ b).real
        return out
    n0, n1, n2 = rho.shape
    flat = rho.reshape(n0 * n1, n2)
    for ia in range(case["n_rad"]):                         # a shell: all (polar, azimuth)
        keep = inside[ia].any(axis=1)
        if not keep.any():
            continue
        sel = torch.from_numpy(np.nonzero(keep)[0]).cuda()
        ez = phases(dev[2][ia, sel, 0], x[2])               # [b, z]: k_z is the ring's
        ex = phases(dev[0][ia, sel], x[0])                  # [b, azi, x]
        ey = phases(dev[1][ia, sel], x[1])
        cc = cd[ia, sel]
        nb = sel.numel()
        step = max(1, int(2.0e8 // (16 * n0 * n1)))         # rings at a time
        for s in range(0, nb, step):
            e = min(nb, s + step)
            z = ez[s:e]
            zr, zi = z.real.t().contiguous(), z.imag.t().contiguous()
            t = torch.complex(flat @ zr, -(flat @ zi))      # [x y, b]: sum over z of rho exp(-i kz z)
            t = t.t().reshape(e - s, n0, n1).contiguous()
            yc = ey[s:e].conj().transpose(1, 2).contiguous()             # [b, y, azi]
            v = torch.bmm(t, yc)                            # [b, x, azi]
            v = (v * ex[s:e].conj().transpose(1, 2)).sum(1)  # [b, azi]
            g = cc[s:e] * cell * v
            p = torch.bmm((g.unsqueeze(1) * ex[s:e].transpose(1, 2)).contiguous(), ey[s:e].contiguous())  # [b, x, y]
            p = p.reshape(e - s, n0 * n1).t()
            out += (p.real.contiguous() @ z.real.contiguous() - p.imag.contiguous() @ z.imag.contiguous()).reshape(
                n0, n1, n2)
    return out


def _short_range(case, axis, rho):
    """I_1 of Eq. 3.9: the padded FFT times (1 - q) Uhat, Nyquist planes left out."""
    dim, shape = case["dim"], _shape(case)
    s, _ = _split_parameters(case)
    pad = [2 * v for v in shape]
    F = torch.fft.fftn(rho.double(), s=pad)
    k = [2.0 * math.pi * torch.fft.fftfreq(p, d=2.0 * L / n, dtype=torch.float64, device="cuda")
         for p, n, L in zip(pad, shape, _box(case))]
    k = [_along(v, i, dim) for i, v in enumerate(k)]
    u = sum(v * v for v in k)
    kn = sum(v * a for v, a in zip(k, axis))
    us = torch.where(u > 0.0, u, torch.ones_like(u))
    if dim == 3:
        mult = -torch.expm1(-u / (s * s)) * (3.0 * kn * kn / us - sum(a * a for a in axis))
    else:
        mult = torch.erf(torch.sqrt(u) / s) * 1.5 * (kn * kn - axis[2] ** 2 * u) / torch.sqrt(us)
    mult = torch.where(u > 0.0, mult, torch.zeros_like(u))
    for i, n in enumerate(shape):
        mult.index_fill_(i, torch.tensor([n], device="cuda"), 0.0)
    out = torch.fft.ifftn(F * mult).real
    return out[tuple(slice(0, n) for n in shape)].contiguous()


def _phi(case, axis, rho):
    out = _direct(case, axis, rho)
    return out + _short_range(case, axis, rho) if case["split"] else out


def _mu2(case):
    dim = case["dim"]
    return sum(_along((math.pi / L * torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device="cuda")) ** 2, i, dim)
               for i, (n, L) in enumerate(zip(_shape(case), _box(case))))


def _trap(case):
    dim = case["dim"]
    return sum(_along(0.5 * (g * x) ** 2, i, dim) for i, (g, x) in enumerate(zip(_gamma(case), _axes(case))))


def exact(case, seed):
    inp = _inputs(case, seed)
    op, axis = case["op"], inp["axis"]
    shape = _shape(case)
    cell = math.prod(2.0 * L / n for n, L in zip(shape, _box(case)))
    if op == "apply":
        return _phi(case, axis, inp["rho"])
    if op == "grad":
        return _phi(case, axis, inp["rho"]), _phi(case, axis, inp["g"])
    if op == "filter":
        return _direct(case, axis, inp["rho"], factors=lambda kk: _yukawa(kk) * 1e-3)
    psi = inp["psi"].to(torch.complex128)
    mu2 = _mu2(case)
    if op == "dynamics":
        kin = torch.polar(torch.ones_like(mu2), -0.25 * _DT_DYN * mu2)
        p1 = torch.fft.ifftn(kin * torch.fft.fftn(psi))
        r1 = p1.real ** 2 + p1.imag ** 2
        th = _DT_DYN * (_trap(case) + _BETA * r1 + _LAM * _phi(case, inp["axis2"], r1))
        p2 = p1 * torch.polar(torch.ones_like(th), -th)
        return torch.fft.ifftn(kin * torch.fft.fftn(p2))
    rho = psi.real ** 2 + psi.imag ** 2
    phi = _phi(case, axis, rho)
    V = _trap(case)
    if op == "energy":
        ph = torch.fft.fftn(psi)
        parts = [0.5 * cell / rho.numel() * float((mu2 * (ph.real ** 2 + ph.imag ** 2)).sum()),
                 cell * float((V * rho).sum()), 0.5 * _BETA * cell * float((rho * rho).sum()),
                 0.5 * _LAM * cell * float((phi * rho).sum())]
        E = np.array(parts + [sum(parts)])
        G = cell * (torch.fft.ifftn(0.5 * mu2 * ph) + (V + _BETA * rho + _LAM * phi) * psi)
        return E, G
    B = V + _BETA * rho + _LAM * phi
    alpha = 0.5 * (B.max() + B.min())
    rhs = torch.fft.fftn(psi) / _DT_FLOW
    den = 1.0 / _DT_FLOW + alpha + 0.5 * mu2
    cur = psi
    for _ in range(case["n_inner"]):
        cur = torch.fft.ifftn((rhs + torch.fft.fftn((alpha - B) * cur)) / den)
    return cur / torch.sqrt(cell * (cur.real ** 2 + cur.imag ** 2).sum())
