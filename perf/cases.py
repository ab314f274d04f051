"""What is timed on an MI355X: the work that a user of this package has it do.

Every case goes through the package's public calls (paper_1412_8250_amd), on the synthetic aluminium cells
of its own input recipes.  listed() names the cases, draw() gives further ones of the same ranges,
prepare() builds what a user's program holds before the call (device arrays, solver contexts), run() is one
pass, work() what a pass cannot do without and exact() the same outputs in 64 bits by other means (spectral
solves with the operator's exact symbol, plain shifts for the stencil, a plain FP64 network).

Paths:
  apply       y = alpha L_h x + beta y, one launch: the smallest call (a 4-atom cell) up to the large cell
  poisson     -L_h phi = 4 pi (rho + b) from zero: plain FP64 CG, FP32 CG in FP64 refinement, multigrid CG
  shifted     the batched complex shifted systems of the kernel terms on cells of different sizes
  multishift  the shifts of one right-hand side by one Krylov sequence
  network     forward and backward of the learned solver aid for one training pair
  scf         whole fixed-point steps from a stored state
"""
import math

import numpy as np
import torch

import paper_1412_8250_amd as ofd
from paper_1412_8250_amd import inputs

RADIUS = 6
A_AL = inputs.A_AL
ALPHA = 5.0 / 6.0 + 5.0 ** 0.5 / 6.0          # the kernel's density powers
BETA = 5.0 / 6.0 - 5.0 ** 0.5 / 6.0
K00 = (complex(-1.68, -1.66), complex(0.236, -0.926), complex(-1.68, 1.66), complex(0.236, 0.926))
DTYPES = {"f64": torch.float64, "f32": torch.float32, "c128": torch.complex128, "c64": torch.complex64}
SIZES = {"f64": 8, "f32": 4, "c128": 16, "c64": 8}
MODES = {"plain": ofd.PLAIN_F64, "refined": ofd.REFINED_F32, "multigrid": ofd.MULTIGRID}


def listed():
    return [
        # one stencil application on the 4-atom cell: launch latency is all there is
        dict(name="apply_f64_16", path="apply", nx=16, ny=16, nz=16, dtype="f64", alpha=1.0, beta=0.0),
        # a complex residual update r = f - A x on a box whose axes fit no tile
        dict(name="apply_c128_ragged", path="apply", nx=110, ny=75, nz=91, dtype="c128", alpha=1.0, beta=1.0),
        # one application on the 16384-atom cell: the bandwidth-bound end
        dict(name="apply_f64_320", path="apply", nx=320, ny=320, nz=320, dtype="f64", alpha=1.0, beta=0.0),
        # the 4-atom cell's electrostatics by the default solver, as its SCF loop and small scans call it
        dict(name="poisson_plain_16", path="poisson", nx=16, ny=16, nz=16, mode="plain", tol=1e-10),
        # a slab-like cell whose axes do not halve: the form for grids that multigrid refuses
        dict(name="poisson_refined_ragged", path="poisson", nx=75, ny=110, nz=54, mode="refined", tol=1e-10),
        # the electrostatics of the 500-atom cell
        dict(name="poisson_multigrid_96", path="poisson", nx=96, ny=96, nz=96, mode="multigrid", tol=1e-10),
        # the electrostatics of the 16384-atom cell
        dict(name="poisson_multigrid_320", path="poisson", nx=320, ny=320, nz=320, mode="multigrid", tol=1e-10),
        # uneven batch: cells of 24^3 .. 96^3 with eight shifts each, no preconditioner
        dict(name="shifted_uneven", path="shifted", cells=6, shifts=8, nmin=24, nmax=96, precond="none",
             dtype="c128", tol=1e-10),
        # the kernel's shifted systems of two 500-atom cells, preconditioned
        dict(name="shifted_multigrid_96", path="shifted", cells=2, shifts=4, nmin=96, nmax=96,
             precond="multigrid", dtype="c128", tol=1e-10),
        # all shifts of one right-hand side on a ragged box
        dict(name="multishift_ragged", path="multishift", nx=130, ny=110, nz=125, shifts=4, tol=1e-10),
        # one training pair of the learned aid on a 64^3 training cell
        dict(name="network_64", path="network", nx=64, ny=64, nz=64),
        # the first fixed-point step of the 16384-atom cell: density update, Poisson, shifted solves, mixing
        dict(name="scf_step_320", path="scf", n=320, form="potential", mu=1, steps=1, sigma=0.8, tol=1e-8),
    ]


def _axis(rng, lo, hi):
    """A grid axis between lo and hi, uniform in its logarithm where the range is wide."""
    if hi > 10 * lo:
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return rng.randint(lo, hi)


def draw(rng):
    path = rng.choice(["apply", "apply", "poisson", "poisson", "poisson", "shifted", "shifted", "multishift",
                       "network", "scf"])
    if path == "apply":
        dt = rng.choice(["f64", "f64", "f32", "c128", "c64"])
        return dict(path=path, nx=_axis(rng, 13, 320), ny=_axis(rng, 13, 320), nz=_axis(rng, 13, 320), dtype=dt,
                    alpha=rng.choice([1.0, -1.0]), beta=rng.choice([0.0, 0.0, 1.0]))
    if path == "poisson":
        mode = rng.choice(["plain", "refined", "multigrid", "multigrid"])
        if mode == "multigrid":                # every axis halves evenly down to at most 16 points
            k = rng.randint(1, 4)
            nx, ny, nz = (rng.randint(9, 16) << k for _ in range(3))
        else:
            nx, ny, nz = (rng.randint(14, 112) for _ in range(3))
        return dict(path=path, nx=nx, ny=ny, nz=nz, mode=mode, tol=1e-10)
    if path == "shifted":
        pre = rng.choice(["none", "multigrid"])
        dt = rng.choice(["c128", "c128", "c64"]) if pre == "none" else "c128"
        nmin = 8 * rng.randint(3, 10)
        return dict(path=path, cells=rng.randint(1, 6), shifts=rng.randint(2, 8), nmin=nmin,
                    nmax=rng.randint(nmin // 8, 12) * 8, precond=pre, dtype=dt, tol=1e-10)
    if path == "multishift":
        return dict(path=path, nx=rng.randint(24, 160), ny=rng.randint(24, 160), nz=rng.randint(24, 160),
                    shifts=rng.randint(2, 8), tol=1e-10)
    if path == "network":
        return dict(path=path, nx=8 * rng.randint(4, 12), ny=8 * rng.randint(4, 12), nz=8 * rng.randint(4, 12))
    form = rng.choice(["potential", "kernel"])
    mu = rng.choice([0, 1])
    # the kernel-potential form solves two Poisson problems per density iteration: smaller cells
    n = rng.choice([32, 48, 64]) if form == "kernel" else rng.choice([32, 48, 64, 80, 96, 128, 160])
    return dict(path=path, n=n, form=form, mu=mu, steps=1, sigma=1.2, tol=1e-8)


# -------------------------------------------------------------------------------------------------------------
# Inputs
# -------------------------------------------------------------------------------------------------------------
_DEV = "cuda"


def _cell(nx, ny, nz, rng, jitter=0.05):
    """FCC cells of 7.5 bohr, as many per axis as keep the spacing near 0.39 bohr."""
    m = [max(1, int(round(k * 0.385 / A_AL))) for k in (nx, ny, nz)]
    atoms = inputs.fcc_atoms(m, A_AL, jitter, rng)
    return inputs.Cell((nx, ny, nz), tuple(A_AL * k for k in m), atoms)


def _densities(cell, rng, sigma=0.8):
    """Nuclear charge b and a smooth electron density rho that balances it (device FP64)."""
    b = inputs.pseudocharge_torch(cell, _DEV, sigma)
    return b, inputs.electron_density_torch(cell, b, rng, _DEV)


def _generator(seed):
    g = torch.Generator(device=_DEV)
    g.manual_seed(int(seed))
    return g


def _weights_1d(h):
    """FD weights w_0 .. w_6 of one axis of spacing h (order 12)."""
    n = RADIUS
    w = [-sum(1.0 / q ** 2 for q in range(1, n + 1)) * 2.0 / h ** 2]
    f = math.factorial
    for p in range(1, n + 1):
        w.append(2.0 * (-1) ** (p + 1) * f(n) ** 2 / (h * h * p * p * f(n - p) * f(n + p)))
    return w


def _laplacian(x, h):
    """L_h x by plain periodic shifts, [nz][ny][nx]."""
    out = torch.zeros_like(x)
    for axis, ha in ((2, h[0]), (1, h[1]), (0, h[2])):
        w = _weights_1d(ha)
        out += w[0] * x
        for p in range(1, RADIUS + 1):
            out += w[p] * (torch.roll(x, p, axis) + torch.roll(x, -p, axis))
    return out


def _symbol(n, h):
    """Eigenvalues of -L_h on the discrete Fourier modes, [nz][ny][nx]."""
    axes = []
    for na, ha in zip(n, h):
        w = _weights_1d(ha)
        k = 2.0 * math.pi * torch.arange(na, dtype=torch.float64, device=_DEV) / na
        # written with sin^2 so that small wave numbers keep their digits: the weights sum to zero
        axes.append(sum(4.0 * w[p] * torch.sin(0.5 * p * k) ** 2 for p in range(1, RADIUS + 1)))
    return axes[2][:, None, None] + axes[1][None, :, None] + axes[0][None, None, :]


def _apply_inputs(case, seed):
    rng = np.random.default_rng([1, seed])
    cell = _cell(case["nx"], case["ny"], case["nz"], rng)
    gen = _generator(seed)
    x = 1.0 + 0.1 * torch.randn(cell.shape, dtype=torch.float64, device=_DEV, generator=gen)
    y = torch.randn(cell.shape, dtype=torch.float64, device=_DEV, generator=gen)
    if case["dtype"] in ("c128", "c64"):
        x = torch.complex(x, torch.randn(cell.shape, dtype=torch.float64, device=_DEV, generator=gen))
        y = torch.complex(y, 0.5 * y)
    dt = DTYPES[case["dtype"]]
    return cell, x.to(dt), y.to(dt)


def _poisson_inputs(case, seed):
    rng = np.random.default_rng([2, seed])
    cell = _cell(case["nx"], case["ny"], case["nz"], rng)
    b, rho = _densities(cell, rng)
    return cell, 4.0 * math.pi * (rho + b)


def _shifted_inputs(case, seed):
    """[(cell, kappa, f)] of every system, system after system of each cell."""
    out = []
    sizes = np.random.default_rng([3, case["cells"], case["nmin"], case["nmax"]])
    for c in range(case["cells"]):
        n = int(sizes.choice(np.arange(case["nmin"], case["nmax"] + 1, 8)))
        rng = np.random.default_rng([3, seed, c])
        cell = _cell(n, n, n, rng)
        _, rho = _densities(cell, rng)
        kappa, factor = inputs.shifted_system_draws(rng, case["shifts"])
        base = (-_laplacian(rho ** ALPHA, cell.h), rho ** BETA)
        for j in range(case["shifts"]):
            f = base[0] if 2 * j < case["shifts"] else base[1]
            out.append((cell, complex(kappa[j]), f.to(torch.complex128) * complex(factor[j])))
    return out


def _multishift_inputs(case, seed):
    rng = np.random.default_rng([4, seed])
    cell = _cell(case["nx"], case["ny"], case["nz"], rng)
    _, rho = _densities(cell, rng)
    extra, _ = inputs.shifted_system_draws(rng, case["shifts"])
    kappas = (list(K00) + [complex(k) for k in extra])[: case["shifts"]]
    return cell, kappas, (-_laplacian(rho ** ALPHA, cell.h)).to(torch.complex128)


def _network_inputs(case, seed):
    """A right-hand side, its solution and He-normal weights."""
    rng = np.random.default_rng([5, seed])
    cell = _cell(case["nx"], case["ny"], case["nz"], rng, jitter=0.1)
    b, rho = _densities(cell, rng)
    g = 4.0 * math.pi * (rho + b)
    g = g - g.mean()
    phi = _solve(g, cell, 0.0).real.contiguous()
    weights = {name: rng.normal(0.0, math.sqrt(2.0 / (27 * ci)), size=(27, ci, co)).astype(np.float32)
               for name, ci, co in ofd.NN_LAYERS}
    return cell, g, phi, weights


def _solve(f, cell, kappa):
    """(-L_h + kappa)^-1 f by the discrete Fourier transform (kappa = 0: zero mean)."""
    sym = _symbol(cell.n, cell.h) + kappa
    fh = torch.fft.fftn(f.to(torch.complex128))
    if kappa == 0.0:
        sym[0, 0, 0] = 1.0
        fh[0, 0, 0] = 0.0
    return torch.fft.ifftn(fh / sym)


# -------------------------------------------------------------------------------------------------------------
# prepare and run
# -------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    path = case["path"]
    if path == "apply":
        cell, x, y = _apply_inputs(case, seed)
        return dict(case=case, h=cell.h, x=x, y0=y, y=torch.empty_like(x))
    if path == "poisson":
        cell, g = _poisson_inputs(case, seed)
        return dict(case=case, solver=ofd.PoissonSolver(cell.shape, cell.h, RADIUS, MODES[case["mode"]]), g=g)
    if path == "shifted":
        systems = _shifted_inputs(case, seed)
        dt = ofd.C128 if case["dtype"] == "c128" else ofd.C64
        batch = ofd.HelmholtzBatch([c.shape for c, _, _ in systems], [c.h for c, _, _ in systems], RADIUS, dt)
        if case["precond"] == "multigrid":
            batch.set_preconditioner(ofd.PRECOND_MULTIGRID)
        return dict(case=case, batch=batch, kappas=[k for _, k, _ in systems], rhs=[f for _, _, f in systems])
    if path == "multishift":
        cell, kappas, f = _multishift_inputs(case, seed)
        solver = ofd.MultiShift(cell.shape, cell.h, RADIUS, max_shifts=len(kappas))
        return dict(case=case, solver=solver, kappas=kappas, f=f)
    if path == "network":
        cell, g, phi, weights = _network_inputs(case, seed)
        net = ofd.Network(1)
        net.set_weights(weights)
        net.set_loss(ofd.Network.ENERGY)
        return dict(case=case, net=net, g=g, phi=phi, h=cell.h)
    # the density update's own tolerance is looser: on the largest cells its residual levels off near 1e-8
    rng = np.random.default_rng([6, seed])
    n = case["n"]
    cell = _cell(n, n, n, rng)
    b, rho = _densities(cell, rng, case["sigma"])
    kernel = case["form"] == "kernel"
    scf = ofd.SCF(cell.shape, cell.h, b, rho.sqrt(), cell.n_electrons, lam=1.0, mu=case["mu"],
                  history=3 if kernel else 7, zeta=1.0 if kernel else 0.3, u_tol=5.0 * case["tol"], u_max_iter=300,
                  poisson_tol=case["tol"], helmholtz_tol=case["tol"], poisson_mode=ofd.MULTIGRID,
                  helmholtz_precond=ofd.PRECOND_MULTIGRID, u_precond=ofd.PRECOND_MULTIGRID, line_slope_tol=1e-2,
                  allow_not_converged=True,
                  fixed_point=ofd.SCF.KERNEL_POTENTIAL if kernel else ofd.SCF.POTENTIAL)
    return dict(case=case, scf=scf, start=scf.snapshot(),
                out={k: torch.empty(cell.shape, dtype=torch.float64, device=_DEV) for k in ("v", "u", "phi")})


def run(state):
    case = state["case"]
    path = case["path"]
    if path == "apply":
        y = state["y"]
        if case["beta"] != 0.0:
            y.copy_(state["y0"])
        return ofd.fd_laplacian_apply(state["x"], y, state["h"], RADIUS, alpha=case["alpha"], beta=case["beta"])
    if path == "poisson":
        phi = torch.zeros_like(state["g"])
        state["solver"].solve(state["g"], phi, case["tol"])
        return phi
    if path == "shifted":
        xs = [torch.zeros_like(f) for f in state["rhs"]]
        state["batch"].solve(state["kappas"], state["rhs"], xs, case["tol"])
        return xs
    if path == "multishift":
        xs = [torch.empty_like(state["f"]) for _ in state["kappas"]]
        state["solver"].solve(state["kappas"], state["f"], xs, case["tol"])
        return xs
    if path == "network":
        loss = state["net"].gradients(state["g"], state["phi"], state["h"])
        return dict(loss=loss, gradients=state["net"].get_weights(gradients=True))
    scf, out = state["scf"], state["out"]
    scf.restore(state["start"])
    for _ in range(case["steps"]):
        scf.step(allow_not_converged=True)
    scf.get(ofd.SCF.V, out["v"])
    scf.get(ofd.SCF.U, out["u"])
    scf.get(ofd.SCF.PHI, out["phi"])
    return out


# -------------------------------------------------------------------------------------------------------------
# work and exact
# -------------------------------------------------------------------------------------------------------------
def work(case):
    """Bytes and operations of one pass.  A Krylov iteration cannot keep its vectors on the chip between its
    two inner products, so the solves count, per iteration, the least vector traffic of their method (each
    vector read and written once per sweep), for the iterations that the method takes on these cells."""
    path = case["path"]
    if path == "scf":
        n = case["n"] ** 3
        # density update ~80 iterations of 3 sweeps, one Poisson solve, four shifted solves, mixing
        per_point = 80 * (24 + 24 + 40 + 16) + 15 * 80 + (4 * 16 * 112 if case["mu"] else 0)
        inner = 26 * 80 * 40 if case["form"] == "kernel" else 0
        return dict(bytes=float(n * (per_point + inner)), flops=float(n * (80 * 150 + 15 * 120)))
    if path == "network":
        n = case["nx"] * case["ny"] * case["nz"]
        per = {"c0a": 1.0, "c0b": 1.0, "d0a": 1.0, "d0b": 1.0, "out": 1.0, "c1a": 1 / 8, "c1b": 1 / 8, "d1a": 1 / 8,
               "d1b": 1 / 8, "c2a": 1 / 64, "c2b": 1 / 64, "d2a": 1 / 64, "d2b": 1 / 64, "c3a": 1 / 512, "c3b": 1 / 512}
        macs = sum(27 * ci * co * per[name] for name, ci, co in ofd.NN_LAYERS)
        acts = sum((ci + co) * per[name] for name, ci, co in ofd.NN_LAYERS)
        return dict(bytes=float(n * (3 * 2 * acts + 24)), flops=float(6 * n * macs))
    if path == "shifted":
        sizes = np.random.default_rng([3, case["cells"], case["nmin"], case["nmax"]])
        n = sum(int(sizes.choice(np.arange(case["nmin"], case["nmax"] + 1, 8))) ** 3 for _ in range(case["cells"]))
        n *= case["shifts"]
        its = 16 if case["precond"] == "multigrid" else 100
        e = 16 if case["dtype"] == "c128" else 8
        return dict(bytes=float(n * its * 7 * e), flops=float(n * its * 120))
    n = case["nx"] * case["ny"] * case["nz"]
    if path == "apply":
        e = SIZES[case["dtype"]]
        c = 2 if case["dtype"].startswith("c") else 1
        return dict(bytes=float(n * e * (3 if case["beta"] else 2)), flops=float(n * c * 55))
    if path == "multishift":
        return dict(bytes=float(n * 60 * 16 * (4 + 3 * case["shifts"])), flops=float(n * 60 * (110 + 16 * case["shifts"])))
    longest = max(case["nx"], case["ny"], case["nz"])
    if case["mode"] == "multigrid":
        return dict(bytes=float(n * 15 * 80), flops=float(n * 15 * 120))
    e = 4 if case["mode"] == "refined" else 8
    its = 4 * longest
    return dict(bytes=float(n * its * 8 * e), flops=float(n * its * 70))


def _network_exact(cell, g, phi, weights):
    """Loss (energy norm) and weight gradients of the U-Net in FP64: 27 shifted matrix products per layer."""
    w = {k: torch.from_numpy(v).to(_DEV).double().requires_grad_(True) for k, v in weights.items()}

    def conv(x, name):
        wt, out, t = w[name], None, 0
        for dz in (-1, 0, 1):
            for dy in (-1, 0, 1):
                for dx in (-1, 0, 1):
                    part = torch.roll(x, (-dz, -dy, -dx), (0, 1, 2)) @ wt[t]
                    out = part if out is None else out + part
                    t += 1
        return out

    def layer(x, name):
        return torch.relu(conv(x, name))

    def pool(x):
        a, b, c, ch = x.shape
        return x.reshape(a // 2, 2, b // 2, 2, c // 2, 2, ch).mean((1, 3, 5))

    def up(x):
        return x.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)

    rms = g.square().mean().sqrt()
    h2 = float(np.cbrt(cell.h[0] * cell.h[1] * cell.h[2])) ** 2
    s0 = layer(layer((g / rms)[..., None], "c0a"), "c0b")
    s1 = layer(layer(pool(s0), "c1a"), "c1b")
    s2 = layer(layer(pool(s1), "c2a"), "c2b")
    d = layer(layer(pool(s2), "c3a"), "c3b")
    d = layer(layer(torch.cat([up(d), s2], -1), "d2a"), "d2b")
    d = layer(layer(torch.cat([up(d), s1], -1), "d1a"), "d1b")
    d = layer(layer(torch.cat([up(d), s0], -1), "d0a"), "d0b")
    out = conv(d, "out")[..., 0]
    t = phi / (h2 * rms)
    e = out - t
    loss = (e * (-h2 * _laplacian(e, cell.h))).sum() / (t * (-h2 * _laplacian(t, cell.h))).sum()
    loss.backward()
    return dict(loss=float(loss), gradients={k: v.grad for k, v in w.items()})


def exact(case, seed):
    path = case["path"]
    if path == "apply":
        cell, x, y = _apply_inputs(case, seed)
        wide = torch.complex128 if x.is_complex() else torch.float64
        out = case["alpha"] * _laplacian(x.to(wide), cell.h)
        return out + case["beta"] * y.to(wide) if case["beta"] != 0.0 else out
    if path == "poisson":
        cell, g = _poisson_inputs(case, seed)
        return _solve(g, cell, 0.0).real.contiguous()
    if path == "shifted":
        return [_solve(f, cell, kappa) for cell, kappa, f in _shifted_inputs(case, seed)]
    if path == "multishift":
        cell, kappas, f = _multishift_inputs(case, seed)
        return [_solve(f, cell, kappa) for kappa in kappas]
    if path == "network":
        return _network_exact(*_network_inputs(case, seed))
    return None          # a whole step has no closed form
