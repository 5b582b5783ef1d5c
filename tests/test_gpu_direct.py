"""The direct solve of the finest level (transforms over x and y, tridiagonal
systems over z) against the oracle's exact discrete solution, on grids that
take each radix of the transforms (8, 4, 2 and odd primes), partial workgroups,
every segment length of the tridiagonal pass and every pair of z faces; and
the multigrid paths it stands in front of, which a context with a multigrid
depth or PIC_FLAG_MG_ALL_LEVELS still takes.

Bounds: FP64 rounding of a length-n transform and of recurrences over nz
planes leaves a relative error of about eps * nz^2 / 10 at most (the condition
number of the z operator times eps); 1e-10 covers nz up to 2000."""
import numpy as np
import pytest

import workloads as W
from oracle import poisson as P

pytestmark = pytest.mark.gpu

BCS = [(0, 0), (1, 0), (0, 1)]
GRIDS = [(2, 2, 2), (4, 2, 4), (16, 8, 24), (40, 20, 36), (96, 48, 62), (14, 22, 10),
         (6, 34, 130), (64, 32, 128), (128, 128, 16), (256, 16, 32), (16, 512, 8),
         (8, 8, 258), (8, 16, 1026), (4, 4, 1500)]


def _case(n, bc, seed):
    p = W.scaled(W.config("c2"), n[0], n[1], n[2], n_e=10, n_ion=10, n_n=10)
    p.update(bc_lo=bc[0], bc_hi=bc[1], v_lo=20.0 if bc[0] == 0 else 2e8,
             v_hi=64.0 if bc[1] == 0 else -1e8)
    p["sources"] = {}
    g = P.Grid(p["nx"], p["ny"], p["nz"], p["dx"], p["bc_lo"], p["bc_hi"], p["v_lo"], p["v_hi"])
    rho = np.random.default_rng(seed).standard_normal(g.shape) * 1e6
    return p, g, rho


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("n", GRIDS)
def test_direct_solve_matches_exact(gpu_lib, n, bc, precision):
    from paper_2606_05893_amd import pic as G
    p, g, rho = _case(n, bc, sum(n))
    p["precision"] = precision
    print("case", n, bc, precision, flush=True)
    ref = P.solve_exact(P.rhs_from_density(rho, g), g)
    gpu = G.Pic(p, capacity=(16, 16, 16))
    scale = np.max(np.abs(ref))
    for start in (None, 0.5 * ref + 3.0 * np.random.default_rng(1).standard_normal(g.shape)):
        if start is not None:  # the given potential carries the face values
            start[0] = ref[0] if bc[0] == 0 else start[0]
            start[-1] = ref[-1] if bc[1] == 0 else start[-1]
        phi, info = gpu.poisson_solve(rho, start)
        assert info["converged"] == 1 and info["vcycles"] == 1
        assert info["refinements"] == (1 if precision == "mixed" else 0)
        assert np.max(np.abs(phi.cpu().numpy() - ref)) <= 1e-10 * scale


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(64, 64, 128), (40, 20, 36), (96, 48, 62)])
def test_multigrid_paths_unchanged(gpu_lib, n, precision):
    """A context that asks for a multigrid depth, or for all levels, runs
    V-cycles: the fused smoother against one launch per colour bit for bit, and
    the exact coarse level against the full hierarchy."""
    from paper_2606_05893_amd import pic as G
    p, g, rho = _case(n, (0, 0), 3)
    p["precision"] = precision
    out = {}
    for name, flags, levels in (("all", G.FLAG_MG_ALL_LEVELS, 0),
                                ("plain", G.FLAG_MG_ALL_LEVELS | G.FLAG_PLAIN_SMOOTHER, 0),
                                ("coarse", 0, 16), ("coarse_plain", G.FLAG_PLAIN_SMOOTHER, 16)):
        q = dict(p, mg_levels=levels)
        phi, info = G.Pic(q, capacity=(16, 16, 16), flags=flags,
                          coarse_sweeps=1024).poisson_solve(rho)
        assert info["converged"] == 1 and info["rel_residual"] <= 1e-10
        out[name] = (phi.cpu().numpy(), info["vcycles"])
    for a, b in (("all", "plain"), ("coarse", "coarse_plain")):
        assert out[a][1] == out[b][1] and np.array_equal(out[a][0], out[b][0])
    assert out["coarse"][1] <= out["all"][1]
    ref = P.solve_exact(P.rhs_from_density(rho, g), g)
    for phi, _ in out.values():
        assert np.max(np.abs(phi - ref)) <= 1e-6 * np.max(np.abs(ref))


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("form", ["apart", "odd word", "same array", "overlap"])
def test_caller_arrays(gpu_lib, form, bc, static):
    """The solve reads the caller's density and start and writes its potential
    itself, or works on copies where the arrays overlap or lie on odd 8-byte
    words: the same potential (FP64 rounding apart), in the caller's array and
    in the context, from zero and from a start, also one that needs no
    correction."""
    import ctypes

    import torch
    from paper_2606_05893_amd import pic as G
    p, g, rho = _case((24, 20, 30), bc, 8)
    scale = np.max(np.abs(ref := P.solve_exact(P.rhs_from_density(rho, g), g)))
    n = ref.size
    gpu = G.Pic(p, capacity=(16, 16, 16))
    cfg = G.make_config(p, capacity=(0, 0, 0), queue_capacity=0, max_events=1)
    buf = torch.zeros(3 * n + 64, dtype=torch.float64, device="cuda")
    off = {"apart": (0, n + n % 2), "odd word": (1, n + 2 + (n + 1) % 2),
           "same array": (0, 0), "overlap": (0, n // 2 - n // 2 % 2)}[form]
    a, b = buf[off[0]:off[0] + n], buf[off[1]:off[1] + n]
    for start in (None, 0.3 * ref, ref):
        if start is not None and off[1] < n:
            continue                       # (a start cannot share the density's words)
        b.copy_(torch.full((n,), 7.0) if start is None else torch.tensor(start).reshape(-1))
        a.copy_(torch.tensor(rho).reshape(-1))
        info = G.SolveInfo()
        warm = 0 if start is None else 1
        ptr = [ctypes.c_void_p(t.data_ptr()) for t in (a, b)]
        if static:
            st = G.load_library().poisson_solve_static(
                ctypes.byref(cfg), ptr[0], ptr[1], warm, ctypes.byref(info),
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        else:
            torch.cuda.synchronize()
            st = gpu.lib.poisson_solve(gpu.ctx, ptr[0], ptr[1], warm, ctypes.byref(info))
        torch.cuda.synchronize()
        assert st == 0 and info.converged == 1
        assert info.vcycles == (0 if start is ref else 1)
        phi = b.cpu().numpy().reshape(ref.shape)
        assert np.max(np.abs(phi - ref)) <= 1e-10 * scale, (form, warm)
        for k, face in ((0, bc[0] == 0), (-1, bc[1] == 0)):
            if face:
                assert np.array_equal(phi[k], np.full_like(phi[k], p["v_lo"] if k == 0 else p["v_hi"]))
        if not static:
            assert np.array_equal(gpu.read_fields()[1].cpu().numpy(), phi)
        if form in ("apart", "odd word"):
            assert np.array_equal(a.cpu().numpy().reshape(ref.shape), rho)
