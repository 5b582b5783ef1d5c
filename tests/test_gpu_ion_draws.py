"""The ion processes' cell pass, which drops a trial whose draw lies above a
bound of its probability, against the oracle, which evaluates every trial:
same counts, near-threshold draws and particles, for cross sections whose
bound comes from the pair's speeds (cx_b = 0), from the energy of its largest
rate (cx_b > 0, tight and loose) or that have none (cx_b < 0); cells from
below to above 32 records, planes of a few and of more than 256 and 4096
records.  Velocities and positions within 1e-12 as in the other parity tests
(mixed: the same trials up to FP32 velocities)."""
import numpy as np
import pytest

import workloads as W
from oracle import pic as O
from oracle import poisson as P

from .test_gpu_ionproc import IONP, compare_all, crowded_load, grid_of, make

pytestmark = pytest.mark.gpu

CX = [(3.1622776601683795e-08, 0.0), (3.2e-8, 1e-9), (2.4e-8, 6e-9),
      (3e-8, -1e-9), (0.0, 0.0)]
KEYS = ("recombinations", "ionisations2", "charge_exchanges")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("k", range(len(CX)))
def test_draws_above_the_bound(gpu_lib, precision, k):
    n = (20000, 20000, 16000) if k % 2 else (4000, 3000, 5000)
    p = W.scaled(W.config("c2"), 16, 16, 16, n_e=n[0], n_ion=n[1], n_n=n[2])
    p["preload"]["kT_e_eV"] = 40.0
    p["precision"] = precision
    p["seed"] = 50 + k
    p["sources"] = {}
    p["ion_processes"] = dict(IONP, cx_a=CX[k][0], cx_b=CX[k][1])
    if k == 2:
        p["ion_processes"].update(lotz_a2=0.0, sigma_rec_1eV=1e-16)
    g = grid_of(p)
    gpu = make(p)
    st = O.State(g, seed=p["seed"])
    crowded_load(p, gpu, st, 80 + k, [((1, 2, 3), 10, 11, 11), ((5, 2, 3), 11, 11, 11),
                                      ((9, 9, 9), 1, 1, 0), ((12, 3, 1), 100, 100, 3900),
                                      ((3, 12, 15), 0, 24, 2)])
    phi = P.solve_exact(P.add_boundary_terms(np.zeros(g.shape), g), g)
    gpu.set_phi(phi)
    _, dg = gpu.advance(p["dt"])
    _, do = O.advance(st, p, O.efield(phi, g), p["dt"])
    print({key: (dg[key], do[key]) for key in KEYS}, dg["near_threshold"], flush=True)
    if precision == "fp64":
        assert dg["near_threshold"] == sum(do["near"].values())
        assert dg["ion_starved"] == do["f3_starved"]
        for key in KEYS:
            assert dg[key] == do[key], key
        compare_all(gpu, st, p, 1e-12, k)
    else:
        for key in KEYS:
            assert abs(dg[key] - do[key]) <= max(3, 0.02 * do[key]), key
    if CX[k][0] > 0.0:
        assert do["charge_exchanges"] > 0
