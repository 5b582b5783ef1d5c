"""The ion processes' time follows the events, not the form of the cross
section: with a charge exchange that depends on the energy (cx_b > 0 and < 0)
the pass takes at most twice its time with a constant one of the same size, and
with some hundred times the events (a per cent of the Cu+ a step) at most three
times.  A cell pass that cannot tell which cells may hold an event runs all of
them, four to six times the time.  The best of five steps each."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

CONST = dict(enabled=True, sigma_rec_1eV=1e-24, lotz_a2=4.5e-18, I2_eV=20.29, cx_a=7.1e-10, cx_b=0.0)


def ion_ms(pre, p, proc):
    from paper_2606_05893_amd import pic as G
    q = dict(p, ion_processes=proc)
    gpu = G.Pic(q, capacity=(2_000_000,) * 4, max_events=1 << 20, flags=G.FLAG_CELL_GROUPS)
    for s, v in pre.items():
        gpu.load(s, *v)
    gpu.set_clock(0, sum(v[0].shape[0] for v in pre.values()))
    gpu.set_phi(torch.zeros((p["nz"] + 1, p["ny"], p["nx"]), dtype=torch.float64, device="cuda"))
    gpu.advance(p["dt"])
    best, cx = float("inf"), 0
    for _ in range(5):
        gpu.enable_timing(True)
        cx = gpu.advance(p["dt"])[1]["charge_exchanges"]
        best = min(best, gpu.phase_times()["ion_coll"][0])
    return best, cx


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_time_follows_the_events(gpu_lib, precision):
    p = W.scaled(W.config("c2"), 64, 64, 256, n_e=1_250_000, n_ion=1_250_000, n_n=625_000)
    p.update(sources={}, precision=precision, v_lo=0.0, v_hi=0.0)
    p["collisions"] = dict(p["collisions"], enabled=False)
    pre = W.preload(p, seed=4)
    base, n0 = ion_ms(pre, p, CONST)
    for name, factor, proc in (("cx_b > 0", 2.0, dict(CONST, cx_a=2.4e-9, cx_b=1e-10)),
                               ("cx_b < 0", 2.0, dict(CONST, cx_b=-1e-12)),
                               ("many events", 3.0, dict(CONST, cx_a=3e-8))):
        ms, n = ion_ms(pre, p, proc)
        print(f"{precision} {name}: {ms:.3f} ms, {n} exchanges; constant {base:.3f} ms, {n0}", flush=True)
        assert ms <= factor * base, name
