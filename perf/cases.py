"""What the speed of this framework is measured on.

Each case is work that a user of the library has it do, through the public
calls of paper_2606_05893_amd.pic, at sizes of the repository's own workloads
(workloads.py, bench.py and the tests' ragged grids):

  run       an interval of a small run: `steps` calls of Pic.step, then the
            fields and every particle are read back, as a surface model
            coupled to the plasma does it.  Launch latency.
  step      one Pic.step of a populated grid: the production step.
  advance   `steps` calls of Pic.advance in a field the caller supplies
            (sources, push, collisions, binning; optionally Coulomb
            collisions or the ion processes), then the charge.
  poisson   one field solve rho -> phi, from zero or from a given potential,
            on a context or through the allocation-free entry point.
  forward   one inference of the warm-start network.
  gradient  the loss and the parameter gradient of one training sample.
  debye     the Debye-length check for each of the block sizes asked for.
"""
import math

import numpy as np
import torch

import workloads as W
from paper_2606_05893_amd import pic as G

_E, _ME, _EPS0, _KB = 1.602176634e-19, 9.1093837139e-31, 8.8541878188e-12, 1.380649e-23
_MCU = 63.546 * 1.66053906892e-27
ROWS = 1 << 15  # of the buffers that particles are handed over in


def listed():
    return [
        # The 32x32x64 run from the disk source alone: all launch latency.
        dict(name="run_32x32x64", kind="run", nx=32, ny=32, nz=64, steps=20),
        # The plain FP64 step of the 128x128x512 plasma.
        dict(name="step_128x128x512", kind="step", nx=128, ny=128, nz=512, n_e=10_000_000,
             n_n=5_000_000, precision="fp64"),
        # The particle side of the mixed-precision step.
        dict(name="advance_mixed", kind="advance", nx=128, ny=128, nz=512, n_e=10_000_000,
             n_n=5_000_000, precision="mixed", process="none", steps=4),
        # ... and of the FP64 step with each of the further collision processes.
        dict(name="advance_coulomb", kind="advance", nx=128, ny=128, nz=512, n_e=10_000_000,
             n_n=5_000_000, precision="fp64", process="coulomb", steps=4),
        dict(name="advance_ion_processes", kind="advance", nx=128, ny=128, nz=512,
             n_e=10_000_000, n_n=5_000_000, precision="fp64", process="ion", steps=4),
        # Field solves: a ragged grid with a Neumann cathode, a small grid without a
        # context, the 128x128x512 grid, and the largest grid in the mixed form from
        # the previous potential.
        dict(name="poisson_40x20x36", kind="poisson", nx=40, ny=20, nz=36, bc_lo=1, bc_hi=0,
             precision="fp64", warm=False, static=False),
        dict(name="poisson_static_64x32x128", kind="poisson", nx=64, ny=32, nz=128, bc_lo=0,
             bc_hi=0, precision="fp64", warm=False, static=True),
        dict(name="poisson_128x128x512", kind="poisson", nx=128, ny=128, nz=512, bc_lo=0,
             bc_hi=0, precision="fp64", warm=False, static=False),
        dict(name="poisson_mixed_256x256x1024", kind="poisson", nx=256, ny=256, nz=1024,
             bc_lo=0, bc_hi=0, precision="mixed", warm=True, static=False),
        # The learned start: inference and a training sample on the 128x128x512 grid.
        dict(name="unet_forward", kind="forward", nx=128, ny=128, nz=512),
        dict(name="unet_gradient", kind="gradient", nx=128, ny=128, nz=512, loss="residual"),
        # The resolution check per cell and per 8^3 block of the plasma.
        dict(name="debye_1_8", kind="debye", nx=128, ny=128, nz=512, n_e=10_000_000,
             block_lo=1, block_hi=8, precision="fp64"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, lo, hi):
    """A size of whole quads of cells, log-uniform, every other one a power of two."""
    v = _log(rng, lo, hi)
    return 1 << round(math.log2(v)) if rng.random() < 0.5 else 4 * round(v / 4)


def draw(rng):
    kind = rng.choice(["run", "step", "advance", "advance", "poisson", "poisson", "forward",
                       "gradient", "debye"])
    prec = rng.choice(["fp64", "mixed"])
    if kind in ("forward", "gradient"):
        c = dict(kind=kind, nx=8 * round(_log(rng, 2, 16)), ny=8 * round(_log(rng, 2, 16)),
                 nz=8 * round(_log(rng, 2, 64)))
        if kind == "gradient":
            c["loss"] = rng.choice(["mse", "residual"])
        return c
    if kind == "poisson":
        bc = rng.choice([(0, 0), (0, 0), (1, 0), (0, 1)])
        c = dict(kind=kind, nx=_size(rng, 8, 256), ny=_size(rng, 8, 256), nz=_size(rng, 16, 512),
                 bc_lo=bc[0], bc_hi=bc[1], precision=prec, warm=rng.random() < 0.5)
        c["static"] = c["nx"] * c["ny"] * c["nz"] < 1_000_000 and rng.random() < 0.5
        return c
    if kind == "run":
        return dict(kind=kind, nx=_size(rng, 16, 48), ny=_size(rng, 16, 48),
                    nz=_size(rng, 32, 96), steps=20)
    if kind == "debye":
        nx, ny, nz = (8 * round(_log(rng, 2, 16)) for _ in range(3))
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, n_e=int(_log(rng, 1e4, 1.2 * nx * ny * nz + 1e4)),
                    block_lo=rng.choice([1, 2]), block_hi=rng.choice([4, 8]), precision=prec)
    nx, ny, nz = _size(rng, 16, 128), _size(rng, 16, 128), _size(rng, 32, 512)
    n_e = int(_log(rng, 1e4, max(2e4, 1.2 * nx * ny * nz)))
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, n_e=n_e, n_n=int(n_e * rng.uniform(0.2, 0.7)),
             precision=prec)
    if kind == "step":
        c["precision"] = "fp64"
    else:
        c["process"] = rng.choice(["none", "coulomb", "ion"])
        c["steps"] = 4
    return c


# ---- inputs -----------------------------------------------------------------
def _params(case):
    """The 128x128x512 workload's physics on the case's grid, the evaporation
    low enough that the population stays near the preload over many steps."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    base = W.config("c1" if case["kind"] == "run" else "c2")
    p = W.scaled(base, nx, ny, nz)
    r_max = 0.4 * min(nx, ny) * p["dx"]
    p["sources"] = {k: dict(s, radius=min(s["radius"], r_max)) for k, s in p["sources"].items()}
    if case["kind"] in ("step", "advance"):
        p["sources"]["disk"]["n_n"] = max(20, nx * ny * nz // 2048)
    p["precision"] = case.get("precision", "fp64")
    p["mg_levels"] = 0
    return p


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, n, p):
    box = torch.tensor([p["nx"], p["ny"], p["nz"]], dtype=torch.float64, device="cuda") * p["dx"]
    return torch.rand((n, 3), dtype=torch.float64, device="cuda", generator=g) * box


def _maxwell(g, n, sigma):
    return torch.randn((n, 3), dtype=torch.float64, device="cuda", generator=g) * sigma


def _populate(pic, case, p, g):
    """Electrons at 5 eV, Cu+ at their positions and (not for the Debye check) Cu at
    3000 K; returns the charged species' positions and velocities."""
    n_e, n_n = case["n_e"], case.get("n_n", 0)
    sig_e, sig_n = math.sqrt(5.0 * _E / _ME), math.sqrt(_KB * 3000.0 / _MCU)
    ids = torch.arange(2 * n_e + n_n, dtype=torch.int64, device="cuda")
    pos, ve, vi = _uniform(g, n_e, p), _maxwell(g, n_e, sig_e), _maxwell(g, n_e, sig_n)
    pic.load(G.ELECTRON, pos, ve, ids[:n_e])
    pic.load(G.ION, pos, vi, ids[n_e:2 * n_e])
    if n_n:
        pic.load(G.NEUTRAL, _uniform(g, n_n, p), _maxwell(g, n_n, sig_n), ids[2 * n_e:])
    pic.set_clock(0, 2 * n_e + n_n)
    return pos, ve, vi


def _smooth_noise(g, shape, volts):
    """Noise of a few cells' extent."""
    f = torch.randn(shape, dtype=torch.float64, device="cuda", generator=g)
    for d in range(3):
        f = (torch.roll(f, 1, d) + 2.0 * f + torch.roll(f, -1, d)) / 4.0
    return f * (volts / float(f.std()))


def _unet_input(case, g):
    """A residual's shape (unit RMS) and a potential between the plates."""
    D, H, Wd = case["nz"], case["ny"], case["nx"]
    x = torch.randn((D, H, Wd, 2), dtype=torch.float32, device="cuda", generator=g)
    ramp = torch.arange(D, dtype=torch.float32, device="cuda") / D
    x[..., 1] = ramp[:, None, None] + 0.02 * x[..., 1]
    return x


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind in ("forward", "gradient"):
        D, H, Wd = case["nz"], case["ny"], case["nx"]
        net = G.UNet(D, H, Wd, params=W.unet_init(int(seed) % 1000))
        st = dict(kind=kind, net=net, x=_unet_input(case, g))
        if kind == "gradient":
            net.set_loss(case["loss"])
            st["t"] = torch.randn((D, H, Wd), dtype=torch.float32, device="cuda", generator=g)
        return st
    p = _params(case)
    st = dict(kind=kind, p=p, case=case)
    if kind == "poisson":
        p.update(bc_lo=case["bc_lo"], bc_hi=case["bc_hi"])
        if case["bc_lo"] == 1:
            p["v_lo"] = 2e8
        if case["bc_hi"] == 1:
            p["v_hi"] = -1e8
        shape = (p["nz"] + 1, p["ny"], p["nx"])
        # The net charge of a neutral plasma's noise: a few e per cell.
        st["rho"] = 2e7 * torch.randn(shape, dtype=torch.float64, device="cuda", generator=g)
        st["phi"] = None
        if case["warm"]:
            z = torch.arange(p["nz"] + 1, dtype=torch.float64, device="cuda") / p["nz"]
            top = p["v_hi"] if case["bc_hi"] == 0 else 0.0
            st["phi"] = (top * z)[:, None, None] + _smooth_noise(g, shape, 1.0)
        # Ragged grids stop coarsening early: a well-solved coarsest level.
        st["kw"] = dict(coarse_sweeps=1024)
        if not case["static"]:
            st["pic"] = G.Pic(p, capacity=(64, 64, 64), **st["kw"])
        return st
    p["seed"] = int(seed)
    if kind == "run":
        cap = 1 << 20
        st["pic"] = G.Pic(p, capacity=(1 << 16, cap, 1 << 16))
        return st
    n_e, n_n = case["n_e"], case.get("n_n", 0)
    flags, kw = 0, {}
    if kind == "advance":
        if case["process"] == "coulomb":
            p["coulomb"] = dict(enabled=True, ln_lambda=10.0)
        if case["process"] == "ion":
            p["ion_processes"] = dict(enabled=True, sigma_rec_1eV=1e-24, lotz_a2=4.5e-18,
                                      I2_eV=20.29, cx_a=math.sqrt(5e-19))
        if case["process"] != "none":
            flags = G.FLAG_CELL_GROUPS
    if kind != "debye":
        extra = 2_000_000
        kw = dict(max_events=1 << 22)
        cap = (n_e + extra, n_n + extra + 4000 * p["sources"]["disk"]["n_n"], n_e + extra, extra)
    else:
        p["sources"] = {}
        cap = (n_e, 16, n_e)
    pic = G.Pic(p, capacity=cap, queue_capacity=1 << 10, flags=flags, **kw)
    _populate(pic, case, p, g)
    if kind == "step":
        pic.set_warm_start("extrap")
    if kind == "advance":
        pic.set_phi(_smooth_noise(g, (p["nz"] + 1, p["ny"], p["nx"]), 2.0))
    st["pic"] = pic
    return st


# ---- one pass ---------------------------------------------------------------
def _diag(d):
    """A step's diagnostics without the solver's own account of its work."""
    return {k: v for k, v in d.items() if k != "solve"}


def _hand_over(st, name, d):
    """Particles into the fixed-size buffers of a surface model."""
    if name not in st:
        st[name] = (torch.empty(ROWS, dtype=torch.int64, device="cuda"),
                    torch.empty((ROWS, 6), dtype=torch.float64, device="cuda"))
    i, x = st[name]
    i.fill_(-1)
    x.zero_()
    if n := min(d["n"], ROWS):
        i[:n], x[:n, :3], x[:n, 3:] = d["id"][:n], d["pos"][:n], d["vel"][:n]
    return i, x


def _by_id(st, species):
    pos, vel, ids = st["pic"].read(species)
    o = torch.argsort(ids)
    return _hand_over(st, species, dict(n=ids.shape[0], id=ids[o], pos=pos[o], vel=vel[o]))


def run(state):
    kind, pic = state["kind"], state.get("pic")
    if kind == "forward":
        return state["net"].forward(state["x"])
    if kind == "gradient":
        return state["net"].gradients(state["x"], state["t"])
    if kind == "poisson":
        if state["case"]["static"]:
            return G.poisson_solve_static(state["p"], state["rho"], state["phi"], **state["kw"])[0]
        return pic.poisson_solve(state["rho"], state["phi"])[0]
    if kind == "debye":
        out = []
        for block in (state["case"]["block_lo"], state["case"]["block_hi"]):
            info, lam = pic.debye_check(block)
            out += [info["blocks"], info["checked"], lam]
        return out
    dt = state["p"]["dt"]
    if kind == "step":
        absorbed, diag = pic.step(dt)
        return _hand_over(state, "absorbed", absorbed), _diag(diag)
    if kind == "run":
        for _ in range(state["case"]["steps"]):
            absorbed, diag = pic.step(dt)
        _, phi, e = pic.read_fields()
        return (_hand_over(state, "absorbed", absorbed), _diag(diag), phi, e, _by_id(state, G.ELECTRON),
                _by_id(state, G.NEUTRAL))
    for _ in range(state["case"]["steps"]):
        absorbed, diag = pic.advance(dt)
    pic.deposit()
    return _hand_over(state, "absorbed", absorbed), _diag(diag), pic.read_fields()[0]


# ---- what a pass cannot do without ------------------------------------------
_UNET = ((2, 16, 0), (16, 16, 0), (16, 32, 1), (32, 32, 1), (32, 64, 2), (64, 64, 2),
         (64, 128, 3), (128, 128, 3), (192, 64, 2), (64, 64, 2), (96, 32, 1), (32, 32, 1),
         (48, 16, 0), (16, 16, 0))


def work(case):
    kind, cells = case["kind"], case["nx"] * case["ny"] * case["nz"]
    nodes = cells + case["nx"] * case["ny"]
    if kind in ("forward", "gradient"):
        flops = sum(2 * 27 * ci * co * (cells >> (3 * lv)) for ci, co, lv in _UNET) + 32 * cells
        n_par = sum(27 * ci * co + co for ci, co, _ in _UNET) + 17
        if kind == "forward":
            return dict(bytes=12 * cells + 4 * n_par, flops=flops)
        return dict(bytes=12 * cells + 8 * n_par, flops=3 * flops)
    if kind == "poisson":
        # rho (and the start) read, phi written; a handful of FLOP per node and
        # octave of the transform a direct solution takes.
        octaves = math.log2(case["nx"] * case["ny"])
        return dict(bytes=8 * nodes * (3 if case["warm"] else 2), flops=5 * nodes * (octaves + 2))
    if kind == "debye":
        per = 48 if case["precision"] == "fp64" else 28
        blocks = sum(cells // b ** 3 for b in (case["block_lo"], case["block_hi"]))
        return dict(bytes=2 * 2 * case["n_e"] * per + 8 * blocks, flops=2 * 2 * case["n_e"] * 12)
    if kind == "run":
        # Per step: the charge read, phi and E written; a few hundred electrons and the
        # evaporated atoms read and written.
        return dict(bytes=case["steps"] * (40 * nodes + 96 * 5000), flops=case["steps"] * 60 * nodes)
    # Positions and velocities read and written, ids read; the cell's field read, the
    # charge written.
    rec = 104 if case["precision"] == "fp64" else 64
    n = 2 * case["n_e"] + case["n_n"]
    b = n * rec + nodes * ((24 if case["precision"] == "fp64" else 12) + 8)
    f = n * 100
    if kind == "step":
        return dict(bytes=b + nodes * 16, flops=f + 60 * nodes)
    if case["process"] != "none":
        b += (2 * case["n_e"] + (case["n_n"] if case["process"] == "ion" else 0)) * 56
        f += 2 * case["n_e"] * 200
    return dict(bytes=case["steps"] * b + 40 * nodes, flops=case["steps"] * f)


# ---- the same in 64 bits ----------------------------------------------------
def _poisson_exact(st):
    """phi on the nodes: real 2-D DFT over x and y, then a tridiagonal elimination over z
    for every mode."""
    p, c = st["p"], st["case"]
    nx, ny, nz, dx = p["nx"], p["ny"], p["nz"], p["dx"]
    b = st["rho"] * (dx * dx / _EPS0)
    k0, k1 = (1 if c["bc_lo"] == 0 else 0), (nz - 1 if c["bc_hi"] == 0 else nz)
    if c["bc_lo"] == 0:
        b[1] += p["v_lo"]
    else:
        b[0] -= 2.0 * dx * p["v_lo"]
    if c["bc_hi"] == 0:
        b[nz - 1] += p["v_hi"]
    else:
        b[nz] += 2.0 * dx * p["v_hi"]
    f = torch.fft.rfft2(b[k0:k1 + 1])
    kx = torch.arange(nx // 2 + 1, dtype=torch.float64, device="cuda")
    ky = torch.arange(ny, dtype=torch.float64, device="cuda")
    d = 6.0 - 2.0 * torch.cos(2 * math.pi * kx / nx)[None] - 2.0 * torch.cos(2 * math.pi * ky / ny)[:, None]
    m = k1 - k0 + 1
    up, inv = [], None
    for k in range(m):  # elimination; a Neumann face's row couples twice to its neighbour
        lo = 0.0 if k == 0 else (2.0 if k == m - 1 and c["bc_hi"] == 1 else 1.0)
        hi = 2.0 if k == 0 and c["bc_lo"] == 1 else 1.0
        inv = 1.0 / (d - lo * up[-1]) if k else 1.0 / d
        if k:
            f[k] += lo * f[k - 1]
        f[k] *= inv
        up.append(hi * inv)
    for k in range(m - 2, -1, -1):
        f[k] += up[k] * f[k + 1]
    phi = torch.empty((nz + 1, ny, nx), dtype=torch.float64, device="cuda")
    phi[k0:k1 + 1] = torch.fft.irfft2(f, s=(ny, nx))
    if c["bc_lo"] == 0:
        phi[0] = p["v_lo"]
    if c["bc_hi"] == 0:
        phi[nz] = p["v_hi"]
    return phi


class _Conv(torch.autograd.Function):
    """3x3x3 convolution of (D, H, W, C), periodic in x and y, zero beyond z."""

    @staticmethod
    def taps(x):
        for dz in (-1, 0, 1):
            a, b = max(0, -dz), x.shape[0] - max(0, dz)
            for dy in (-1, 0, 1):
                for dx in (-1, 0, 1):
                    yield a, b, dz, dy, dx

    @staticmethod
    def forward(ctx, x, w):
        ctx.save_for_backward(x, w)
        out = torch.zeros(x.shape[:3] + (w.shape[0],), dtype=x.dtype, device=x.device)
        for t, (a, b, dz, dy, dx) in enumerate(_Conv.taps(x)):
            out[a:b] += torch.roll(x[a + dz:b + dz], (-dy, -dx), (1, 2)) @ w[:, t].t()
        return out

    @staticmethod
    def backward(ctx, gy):
        x, w = ctx.saved_tensors
        gx, gw = torch.zeros_like(x), torch.zeros_like(w)
        for t, (a, b, dz, dy, dx) in enumerate(_Conv.taps(x)):
            gx[a + dz:b + dz] += torch.roll(gy[a:b] @ w[:, t], (dy, dx), (1, 2))
            xs = torch.roll(x[a + dz:b + dz], (-dy, -dx), (1, 2)).reshape(-1, x.shape[3])
            gw[:, t] = gy[a:b].reshape(-1, gy.shape[3]).t() @ xs
        return gx, gw


def _unet_exact(x, par):
    """The network in float64 from its documented parameter layout."""
    at = 0

    def conv(h, k):
        nonlocal at
        ci, co, _ = _UNET[k]
        w = par[at:at + co * 27 * ci].reshape(co, 27, ci)
        b = par[at + co * 27 * ci:at + co * 27 * ci + co]
        at += co * 27 * ci + co
        return torch.relu(_Conv.apply(h, w) + b)

    def pool(h):
        D, H, Wd, C = h.shape
        return h.reshape(D // 2, 2, H // 2, 2, Wd // 2, 2, C).mean((1, 3, 5))

    def up(h):
        return h.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)

    h0 = conv(conv(x, 0), 1)
    h1 = conv(conv(pool(h0), 2), 3)
    h2 = conv(conv(pool(h1), 4), 5)
    h = conv(conv(pool(h2), 6), 7)
    h = conv(conv(torch.cat([up(h), h2], 3), 8), 9)
    h = conv(conv(torch.cat([up(h), h1], 3), 10), 11)
    h = conv(conv(torch.cat([up(h), h0], 3), 12), 13)
    return h @ par[at:at + 16] + par[at + 16]


def _residual_loss(e):
    """Sum of (A e)^2 over the planes above a Dirichlet cathode, per voxel."""
    z = torch.zeros_like(e[:1])
    u = torch.cat([z, e[1:], z])  # the cathode plane is known, the anode beyond the top
    q = 6.0 * u - torch.roll(u, 1, 1) - torch.roll(u, -1, 1) - torch.roll(u, 1, 2) - torch.roll(u, -1, 2)
    q = q[1:-1] - u[:-2] - u[2:]
    return (q * q).sum() / e.numel()


def _debye_exact(case, pos, ve, vi, block, p):
    nb = [case[k] // block for k in ("nx", "ny", "nz")]
    h = block * p["dx"]
    ijk = (pos / h).floor().to(torch.int64)
    for d in range(3):
        ijk[:, d].clamp_(0, nb[d] - 1)
    key = (ijk[:, 2] * nb[1] + ijk[:, 1]) * nb[0] + ijk[:, 0]
    m = nb[0] * nb[1] * nb[2]
    n = torch.zeros(m, dtype=torch.float64, device="cuda").index_add_(0, key, torch.ones_like(pos[:, 0]))
    inv = torch.zeros_like(n)
    for v, mass in ((ve, _ME), (vi, _MCU)):
        mean = torch.zeros((m, 3), dtype=torch.float64, device="cuda").index_add_(0, key, v) / n[:, None]
        dev = ((v - mean[key]) ** 2).sum(1)
        kt = mass * torch.zeros_like(n).index_add_(0, key, dev) / (3.0 * (n - 1.0))
        inv += torch.where(n >= 2, n / h ** 3 * _E * _E / (_EPS0 * kt), 0.0)
    return (1.0 / torch.sqrt(inv)).reshape(nb[2], nb[1], nb[0])


def exact(case, seed):
    kind = case["kind"]
    if kind == "poisson":
        return _poisson_exact(prepare(dict(case), seed))
    if kind in ("forward", "gradient"):
        x = _unet_input(case, g := _gen(seed)).double()
        par = torch.tensor(np.asarray(W.unet_init(int(seed) % 1000)), dtype=torch.float64, device="cuda")
        if kind == "forward":
            with torch.no_grad():
                return _unet_exact(x, par)
        t = torch.randn(x.shape[:3], dtype=torch.float32, device="cuda", generator=g).double()
        par.requires_grad_(True)
        e = _unet_exact(x, par) - t
        loss = (e * e).mean() if case["loss"] == "mse" else _residual_loss(e)
        loss.backward()
        return par.grad, float(loss.detach())
    if kind == "debye" and case["precision"] == "fp64":
        p, g = _params(case), _gen(seed)
        pos = _uniform(g, case["n_e"], p)
        ve = _maxwell(g, case["n_e"], math.sqrt(5.0 * _E / _ME))
        vi = _maxwell(g, case["n_e"], math.sqrt(_KB * 3000.0 / _MCU))
        out = []
        for block in (case["block_lo"], case["block_hi"]):
            out += [None, None, _debye_exact(case, pos, ve, vi, block, p)]
        return out
    return None  # particles with random collisions have no value in 64 bits
