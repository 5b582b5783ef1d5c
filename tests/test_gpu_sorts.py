"""Record sorts of a step: the cathode list, which every step returns sorted by
(species, id), for lists on both sides of the lengths where the sort changes
its way (known short lengths by rank in one launch, else chunks and merges),
growing and shrinking between steps so that the way chosen by the last length
meets another one, against numpy's sort of the same records."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [(3, 1, 64, 65, 0, 1000), (300, 4096, 4097, 100, 5000),
                                     (8000, 9000, 40000, 100, 70000, 9), (1, 20000, 8192, 8193)])
def test_cathode_list_sorted(gpu_lib, lengths):
    from paper_2606_05893_amd import pic as G
    p = W.scaled(W.config("c2"), 16, 16, 32)
    p["sources"] = {}
    p["collisions"] = dict(p["collisions"], enabled=False)
    gpu = G.Pic(p, capacity=(1 << 17, 1 << 17, 1 << 17), queue_capacity=1 << 17,
                max_events=1 << 17)
    gpu.set_phi(np.zeros((p["nz"] + 1, p["ny"], p["nx"])))
    rng = np.random.default_rng(sum(lengths))
    dt, dx, next_id = p["dt"], p["dx"], 0
    for n in lengths:
        # n particles of two species just above the cathode, falling through it.
        split = int(n * 0.6)
        want = []
        for sp, m in ((G.ION, split), (G.ELECTRON, n - split)):
            if not m:
                continue
            pos = rng.random((m, 3)) * [p["nx"] * dx, p["ny"] * dx, 0.2 * dx]
            vel = np.zeros((m, 3))
            vel[:, 2] = -(pos[:, 2] + 0.5 * dx) / dt
            gpu.inject(sp, pos, vel)
            want += [(sp, next_id + k, vel[k, 2]) for k in range(m)]
            next_id += m
        ab, d = gpu.advance(dt)
        assert ab["n"] == n and d["cathode"][0] + d["cathode"][2] == n
        if n:
            want.sort(key=lambda r: r[:2])
            got = list(zip(ab["species"].tolist(), ab["id"].tolist(), ab["vel"][:, 2].tolist()))
            assert got == want, n
