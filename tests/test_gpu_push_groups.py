"""The tile push at the edges of its split: a tile's ions and electrons go to
the waves 64 at a time and in pieces of 2048, and collision probabilities
come from a table for fewer than 64 neutrals in the cell.  One step from an
identical state against the oracle: particle sets, uncollided trajectories,
the charge of the pushed state and the counts exactly, collided velocities
within 1e-12 (mixed: 1e-4, FP32 offsets and velocities), kinetic sums of at
most 10^4 terms in another order within 1e-12 (mixed 1e-5).
"""
import numpy as np
import pytest

import workloads as W
from oracle import constants as C
from oracle import pic as O
from oracle import poisson as P

pytestmark = pytest.mark.gpu

# Per case: (tile origin cell, electrons, Cu+) for a few tiles, and the
# neutrals of one cell of the first tile.
CASES = [
    ([((0, 0, 0), 0, 1), ((8, 0, 0), 1, 0)], 1),
    ([((0, 0, 0), 63, 64), ((8, 8, 8), 64, 63)], 63),
    ([((0, 0, 0), 65, 65), ((8, 8, 0), 129, 1)], 64),
    ([((0, 8, 8), 255, 257), ((8, 0, 16), 257, 0)], 65),
    ([((8, 8, 16), 2049, 2048), ((0, 0, 8), 0, 2049)], 300),
]


def by_id(pos, vel, ids):
    ids = np.asarray(ids).astype(np.uint64)
    o = np.argsort(ids)
    return ids[o], np.asarray(pos)[o], np.asarray(vel)[o]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("k", range(len(CASES)))
def test_push_groups(gpu_lib, precision, k):
    from paper_2606_05893_amd import pic as G
    tiles, n_cell = CASES[k]
    p = W.scaled(W.config("c2"), 16, 16, 24, n_e=0, n_ion=0, n_n=0)
    p["precision"] = precision
    p["seed"] = 20 + k
    p["sources"] = {}
    p["collisions"] = dict(p["collisions"], sigma_el=3e-17, lotz_a=4.5e-15)
    g = P.Grid(p["nx"], p["ny"], p["nz"], p["dx"], p.get("bc_lo", 0),
               p.get("bc_hi", 0), p.get("v_lo", 0.0), p.get("v_hi", 0.0))
    gpu = G.Pic(p, capacity=(20000, 20000, 20000))
    st = O.State(g, seed=p["seed"])
    rng = np.random.default_rng(30 + k)
    sig = {C.ELECTRON: np.sqrt(10.0 * C.E_CHARGE / C.M_E),
           C.ION: np.sqrt(C.K_B * 3000.0 / C.M_CU)}
    sig[C.NEUTRAL] = sig[C.ION]
    parts = {s: [] for s in sig}
    for org, ne, ni in tiles:
        for s, n in ((C.ELECTRON, ne), (C.ION, ni)):
            parts[s].append((np.array(org) + 8.0 * rng.random((n, 3))) * p["dx"])
    cell = np.array(tiles[0][0]) + 3
    parts[C.NEUTRAL].append((cell + 0.2 + 0.6 * rng.random((n_cell, 3))) * p["dx"])
    parts[C.ELECTRON].append((cell + 0.2 + 0.6 * rng.random((5, 3))) * p["dx"])
    parts[C.NEUTRAL].append(W.random_particles(3000, p, 40 + k)[0])
    nid = 0
    for s in parts:
        pos = np.concatenate(parts[s])
        vel = rng.standard_normal(pos.shape) * sig[s]
        if precision == "mixed":
            vel = vel.astype(np.float32).astype(np.float64)
        ids = np.arange(nid, nid + len(pos), dtype=np.uint64)
        nid += len(pos)
        st.load(s, pos, vel, ids)
        gpu.load(s, pos, vel, ids)
    st.next_id = nid
    gpu.set_clock(0, nid)
    phi = P.solve_exact(P.add_boundary_terms(np.zeros(g.shape), g), g)
    phi = phi + rng.standard_normal(g.shape)
    gpu.set_phi(phi)
    _, dg = gpu.advance(p["dt"])
    _, do = O.advance(st, p, O.efield(phi, g), p["dt"])
    for s in range(3):
        assert dg["cathode"][s] == do["cathode"][s]
        assert dg["anode"][s] == do["anode"][s]
    fp64 = precision == "fp64"
    if fp64:
        assert dg["near_threshold"] == sum(do["near"].values())
        for key in ("candidates", "elastic", "ionisations", "starved"):
            assert dg[key] == do[key], key
    for s in range(3):
        pg, vg, ig = (t.cpu().numpy() for t in gpu.read(s))
        ig, pg, vg = by_id(pg, vg, ig)
        sp = st.sp[s]
        io, po, vo = by_id(np.stack([sp[q] for q in ("x", "y", "z")], 1),
                           np.stack([sp[q] for q in ("vx", "vy", "vz")], 1),
                           sp["id"])
        if fp64:
            assert np.array_equal(ig, io), s
        common, ia, ib = np.intersect1d(ig, io, return_indices=True)
        assert common.size >= 0.999 * io.size
        if not common.size:
            continue
        vs = np.maximum(np.abs(vo[ib]), np.sqrt(np.mean(vo ** 2)))
        tol = 1e-12 if fp64 else 1e-4
        assert np.all(np.abs(vg[ia] - vo[ib]) <= tol * vs), s
        d = np.abs(pg[ia] - po[ib])
        assert np.all(d <= (1e-12 if fp64 else 1e-4) * p["dx"] + 1e-12 * po[ib]), s
        assert np.isclose(dg["kinetic"][s], do["kinetic"][s],
                          rtol=1e-12 if fp64 else 1e-5)
    gpu.deposit()
    acc = gpu.read_fields()[0].cpu().numpy()
    acc_o = O.deposit(st)
    if fp64:
        assert np.array_equal(acc, acc_o)
    else:
        # An FP32 offset moves a weight by at most one of 8192 steps per axis.
        n = len(st.sp[0]["id"]) + len(st.sp[2]["id"])
        assert acc.sum() == acc_o.sum()
        assert np.abs(acc - acc_o).sum() <= n * 8 * 3 * 2 ** 26


@pytest.mark.parametrize("shape", [(8, 8, 8), (16, 8, 504), (120, 72, 136), (256, 256, 256),
                                   (256, 256, 264)])
def test_tile_ranges(gpu_lib, shape):
    """The scan of the tile counts by one workgroup (1 to 32768 tiles) and by
    blocks (beyond): after two steps without field or collisions the binned
    deposit is the oracle's charge bit for bit and no particle is lost."""
    from paper_2606_05893_amd import pic as G
    p = W.scaled(W.config("c2"), *shape, n_e=0, n_ion=0, n_n=0)
    p["sources"] = {}
    p["collisions"] = dict(p["collisions"], enabled=False)
    p.update(v_lo=0.0, v_hi=0.0)
    g = P.Grid(p["nx"], p["ny"], p["nz"], p["dx"], 0, 0, 0.0, 0.0)
    gpu = G.Pic(p, capacity=(9000, 9000, 9000))
    st = O.State(g, seed=1)
    for s, n in ((0, 6000), (2, 5000)):
        pos, vel, ids = W.random_particles(n, p, 60 + s, id0=10000 * s, z_margin=1)
        vel = vel * 0.0 + np.random.default_rng(s).uniform(-0.4, 0.4, vel.shape) * p["dx"] / p["dt"]
        vel[:, 2] *= 0.1
        st.load(s, pos, vel, ids)
        gpu.load(s, pos, vel, ids)
    st.next_id = 30000
    gpu.set_clock(0, 30000)
    gpu.set_phi(np.zeros(g.shape))
    E = np.zeros((3,) + g.shape)
    for _ in range(2):
        _, dg = gpu.advance(p["dt"])
        _, do = O.advance(st, p, E, p["dt"])
        for s in range(3):
            assert dg["counts"][s] == do["counts"][s]
    gpu.deposit()
    assert np.array_equal(gpu.read_fields()[0].cpu().numpy(), O.deposit(st))
    pos, vel, ids = (t.cpu().numpy() for t in gpu.read(0))
    gpu.load(0, pos, vel, ids)          # (binned afresh: a full pass deposits)
    gpu.deposit()
    assert np.array_equal(gpu.read_fields()[0].cpu().numpy(), O.deposit(st))
