"""The Debye-length resolution check on the GPU against the oracle, on the
particle state a step leaves (electrons binned by tile, ions partly in
their unbinned tail), for blocks of 1, 2, 4 and 8 cells per axis: lambda_D
per block within 1e-9 (the moments are summed in another order), the
numbers of checked and unresolved blocks exactly (blocks within 1e-9 of
the criterion excepted), the smallest Debye length and the largest
dx / d_max within 1e-9.  An empty state has nothing to check."""
import numpy as np
import pytest

import workloads as W
from oracle import pic as O
from oracle import poisson as P

pytestmark = pytest.mark.gpu


def _state_pair(precision="fp64"):
    from paper_2606_05893_amd import pic as G
    p = W.scaled(W.config("c2"), 32, 32, 64, n_e=150000, n_ion=150000,
                 n_n=20000)
    p["precision"] = precision
    gpu = G.Pic(p, capacity=(400000, 400000, 400000))
    pre = W.preload(p, seed=31)
    for s, (pos, vel, ids) in pre.items():
        gpu.load(s, pos, vel, ids)
    gpu.set_clock(0, sum(v[0].shape[0] for v in pre.values()))
    gpu.step(p["dt"])
    g = P.Grid(p["nx"], p["ny"], p["nz"], p["dx"], p["bc_lo"], p["bc_hi"],
               p["v_lo"], p["v_hi"])
    st = O.State(g, w_sp=p["w_sp"])
    for s in range(3):
        pos, vel, ids = (t.cpu().numpy() for t in gpu.read(s))
        st.load(s, pos, vel, ids.astype(np.uint64))
    return p, gpu, st


@pytest.mark.parametrize("block", [1, 2, 4, 8])
def test_debye_check_matches_oracle(gpu_lib, block):
    p, gpu, st = _state_pair()
    # alpha_D chosen so that the criterion splits the blocks.
    for alpha in (0.5, 4.0):
        info, lam = gpu.debye_check(block, alpha)
        ref = O.debye_check(st, block, alpha)
        lam = lam.cpu().numpy()
        fin = np.isfinite(ref["lambda_D"])
        assert np.array_equal(np.isfinite(lam), fin)
        assert np.all(np.abs(lam[fin] - ref["lambda_D"][fin])
                      <= 1e-9 * ref["lambda_D"][fin])
        assert info["checked"] == ref["checked"]
        ratio = p["dx"] / (3.4 * alpha * ref["lambda_D"][fin])
        edge = int(np.count_nonzero(np.abs(ratio - 1.0) < 1e-9))
        assert abs(info["unresolved"] - ref["unresolved"]) <= edge
        assert abs(info["lambda_min"] - ref["lambda_min"]) <= 1e-9 * ref["lambda_min"]
        assert abs(info["ratio_max"] - ref["ratio_max"]) <= 1e-9 * ref["ratio_max"]
        print("block", block, "alpha", alpha, info, flush=True)
    assert info["blocks"] == lam.size


def test_debye_check_mixed_and_empty(gpu_lib):
    from paper_2606_05893_amd import pic as G
    p, gpu, st = _state_pair("mixed")
    info, _ = gpu.debye_check(4, 0.5, with_lambda=False)
    ref = O.debye_check(st, 4, 0.5)
    # The read-back positions are (cell + FP32 offset) dx: a particle within
    # rounding of a cell face may land in the neighbouring block.
    assert abs(info["checked"] - ref["checked"]) <= 2
    assert abs(info["lambda_min"] - ref["lambda_min"]) <= 1e-3 * ref["lambda_min"]
    q = W.scaled(W.config("c2"), 16, 16, 16, n_e=1, n_ion=1, n_n=1)
    empty = G.Pic(q, capacity=(16, 16, 16))
    info, lam = empty.debye_check(2, 0.5)
    assert info["checked"] == 0 and info["unresolved"] == 0
    assert np.isinf(info["lambda_min"]) and bool(lam.isinf().all())
    with pytest.raises(G.PicError):
        empty.debye_check(3, 0.5)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", ["ragged", "strays", "crowded"])
def test_debye_tile_and_record_paths(gpu_lib, case, precision):
    """The tile pass on a grid that ends inside its tiles, with ions that left
    their tiles and an unbinned tail (new ions and ions moved by a field over
    steps that do not bin them), and the record path of crowded tiles, against
    the oracle on the particles read back.  The cells of the mixed form are
    exact; its read-back positions may round into the neighbouring cell, so
    its blocks are compared over all of them: counts within 1e-3, and the
    median Debye length within 1e-3."""
    from paper_2606_05893_amd import pic as G
    n = (20, 12, 36) if case != "crowded" else (8, 8, 16)
    npart = 20000 if case != "crowded" else 30000
    p = W.scaled(W.config("c2"), *n, n_e=npart, n_ion=npart, n_n=5000)
    p["precision"] = precision
    r = 0.4 * min(n[0], n[1]) * p["dx"]
    p["sources"] = {k: dict(s, radius=min(s["radius"], r)) for k, s in p["sources"].items()}
    gpu = G.Pic(p, capacity=(400000, 400000, 400000))
    pre = W.preload(p, seed=7)
    for s, (pos, vel, ids) in pre.items():
        if case == "strays" and s == 2:
            vel = vel * 300.0  # a tenth of a cell a step
        gpu.load(s, pos, vel, ids)
    gpu.set_clock(0, sum(v[0].shape[0] for v in pre.values()))
    for _ in range(3 if case == "strays" else 1):
        gpu.step(p["dt"])
    g = P.Grid(p["nx"], p["ny"], p["nz"], p["dx"], p["bc_lo"], p["bc_hi"], p["v_lo"], p["v_hi"])
    st = O.State(g, w_sp=p["w_sp"])
    for s in range(3):
        pos, vel, ids = (t.cpu().numpy() for t in gpu.read(s))
        st.load(s, pos, vel, ids.astype(np.uint64))
    for block in (1, 2, 4, 8):
        if any(d % block for d in n):
            continue
        info, lam = gpu.debye_check(block, 0.5)
        ref = O.debye_check(st, block, 0.5)
        lam = lam.cpu().numpy()
        fin = np.isfinite(ref["lambda_D"])
        print(case, precision, block, info, flush=True)
        if precision == "fp64":
            assert np.array_equal(np.isfinite(lam), fin)
            assert np.all(np.abs(lam[fin] - ref["lambda_D"][fin]) <= 1e-9 * ref["lambda_D"][fin])
            assert info["checked"] == ref["checked"]
        else:
            assert abs(info["checked"] - ref["checked"]) <= 1e-3 * ref["checked"] + 1
            a, b = np.median(lam[np.isfinite(lam)]), np.median(ref["lambda_D"][fin])
            assert abs(a - b) <= 1e-3 * b
