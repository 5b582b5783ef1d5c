"""V-cycles, which a context with a multigrid depth (mg_levels > 0) runs in
poisson_solve, in the allocation-free solve and in its steps, and every context
in steps on fewer than 2^18 nodes: on ragged, unequal and tiny grids, with
Dirichlet and Neumann faces at either end, in FP64 and in the mixed form.

* The fused two-sweep smoothing pass and one launch per colour and sweep are the
  same arithmetic: the same potential and cycle count, bit for bit.
* The exact solve of the first small coarse level (by FFT on powers of two up to
  64, directly on other even axes up to 32) and the cycle down to the coarsest
  level both reach the 1e-10 residual, agree within 1e-8 (the residual bound
  times the operator's condition in these grids) and with the oracle's exact
  solution within 1e-6, and the exact level takes no more cycles.
* The allocation-free solve is the context's, bit for bit, also where its buffer
  holds another grid's values.
* A step's potential is the oracle's within 1e-6.
"""
import numpy as np
import pytest

import workloads as W
from oracle import pic as O
from oracle import poisson as P

from .test_gpu_parity import grid_of, load_both, make

pytestmark = pytest.mark.gpu

BCS = [(0, 0), (1, 0), (0, 1)]
# Levels of 64 x 16 (FP32 32 x 16) columns and more, of 16 x 16 columns, below them
# (one launch per colour), and tiles that end ragged; first coarse levels of 64 x
# 16 and 8 x 4 nodes by FFT, of 20 x 10 directly, and none (the second coarsening
# of 96x48x62 and 136x80x34 stops).
GRIDS = [(64, 64, 128), (40, 20, 36), (96, 48, 62), (128, 32, 40), (16, 8, 24), (32, 32, 64),
         (16, 16, 20), (136, 80, 34)]


def case(n, bc, precision, seed):
    p = W.scaled(W.config("c2"), *n, n_e=10, n_ion=10, n_n=10)
    p.update(bc_lo=bc[0], bc_hi=bc[1], precision=precision, mg_levels=16, sources={})
    if bc[0] == 1:
        p["v_lo"] = -2e8
    if bc[1] == 1:
        p["v_hi"] = 3e8
    rho = np.random.default_rng(seed).standard_normal((n[2] + 1, n[1], n[0])) * 1e6
    return p, rho


def solve(p, rho, flags=0):
    from paper_2606_05893_amd import pic as G
    # Ragged grids stop coarsening early: a well-solved coarsest level.
    gpu = G.Pic(p, capacity=(64, 64, 64), flags=flags, coarse_sweeps=1024)
    phi, info = gpu.poisson_solve(rho)
    assert info["converged"] == 1 and info["rel_residual"] <= 1e-10
    assert info["vcycles"] >= 2  # (a direct solve takes one)
    return phi.cpu().numpy(), info["vcycles"]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("n", GRIDS)
def test_vcycles(gpu_lib, n, bc, precision):
    from paper_2606_05893_amd import pic as G
    p, rho = case(n, bc, precision, sum(n))
    all_, plain = G.FLAG_MG_ALL_LEVELS, G.FLAG_PLAIN_SMOOTHER
    out = {f: solve(p, rho, f) for f in (0, plain, all_, all_ | plain)}
    print(n, bc, precision, {f: v[1] for f, v in out.items()}, flush=True)
    for f in (0, all_):
        assert out[f][1] == out[f | plain][1]
        assert np.array_equal(out[f][0], out[f | plain][0])
    assert out[0][1] <= out[all_][1]
    ref = P.solve_exact(P.rhs_from_density(rho, g := grid_of(p)), g)
    scale = np.max(np.abs(ref))
    assert np.max(np.abs(out[0][0] - out[all_][0])) <= 1e-8 * scale
    for phi, _ in out.values():
        assert np.max(np.abs(phi - ref)) <= 1e-6 * scale


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_static_vcycles(gpu_lib, precision):
    from paper_2606_05893_amd import pic as G
    for n, bc in (((64, 32, 128), (0, 0)), ((32, 16, 32), (1, 0)), ((64, 32, 32), (0, 1))):
        p, rho = case(n, bc, precision, n[2])
        phi, info = G.poisson_solve_static(p, rho, coarse_sweeps=1024)
        ref, cycles = solve(p, rho)
        assert info["converged"] == 1 and info["vcycles"] == cycles
        assert np.array_equal(phi.cpu().numpy(), ref)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("levels", [0, 16])
@pytest.mark.parametrize("bc", BCS)
def test_step(gpu_lib, bc, levels, precision):
    p = W.scaled(W.config("c2"), 32, 16, 24, n_e=4000, n_ion=4000, n_n=3000)
    field = p["v_hi"] / (p["nz"] * p["dx"])
    p.update(bc_lo=bc[0], bc_hi=bc[1], precision=precision, mg_levels=levels, sources={})
    if bc[0] == 1:
        p["v_lo"] = field
    if bc[1] == 1:
        p["v_hi"] = field
    gpu = make(p)
    st = O.State(grid_of(p), seed=3)
    load_both(p, gpu, st, seed=9)
    _, d = gpu.step(p["dt"])
    _, _, phi_o = O.step(st, p, p["dt"])
    phi = gpu.read_fields()[1].cpu().numpy()
    assert d["solve"]["converged"] == 1 and d["solve"]["rel_residual"] <= 1e-10
    assert d["solve"]["vcycles"] >= 2
    assert np.max(np.abs(phi - phi_o)) <= 1e-6 * np.max(np.abs(phi_o))
