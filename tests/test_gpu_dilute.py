"""Lists that need padding where every candidate of the 27 cells is in them: a
dilute gas, and small clusters far apart.  They are padded with a particle from
elsewhere in the replica; only where it has none does the replica stop."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import TOL_F, say
from oracle import oracle as O
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu


def _gas(n, rho):
    """A random subset of the sites of a lattice whose neighbours just touch."""
    box, rng = I.box_length(n, rho), np.random.default_rng(n)
    m = int(box / 4.0 ** (1.0 / 3.0))
    sites = I.fcc_positions(4 * m ** 3, box, None)
    pos = sites[np.sort(rng.choice(len(sites), size=n, replace=False))]
    pos = np.mod(pos + rng.uniform(-0.03, 0.03, pos.shape), box)
    return I.System(n, box, pos, I.maxwell_velocities(n, 1.0, rng), np.zeros(n, dtype=np.int32), I.lj_table(I.WCA_RC), 1.0)


def _clusters(n_clusters, edge):
    """Tight cubes of edge^3 particles, one to every third cell, so that each
    particle's 27 cells hold its own cluster and nothing else."""
    rl, a = 3.0 + 0.3, 0.46
    box = n_clusters * 3.0 * rl + 0.05
    g = np.arange(edge) * a
    cube = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    at = (np.arange(n_clusters) * 3.0 + 1.3) * rl
    centres = np.stack(np.meshgrid(at, at, at, indexing="ij"), -1).reshape(-1, 3)
    pos = (centres[:, None, :] + cube[None, :, :]).reshape(-1, 3)
    n = len(pos)
    t = I.lj_table(3.0)
    t.sigma[:] = 0.4
    return I.System(n, float(np.float32(box)), pos, I.maxwell_velocities(n, 0.01, np.random.default_rng(1)),
                    np.zeros(n, dtype=np.int32), t, 0.01)


SYSTEMS = {
    "gas": lambda: _gas(3000, 0.1),           # 21^3 cells of 0.3
    "thin_gas": lambda: _gas(500, 0.02),      # 20^3 cells of 0.06
    "members": lambda: _gas(20000, 0.05),     # 51^3 cells, a lane per member
    "products": lambda: _clusters(2, 4),      # cells of 64, on the matrix cores
}


@pytest.mark.parametrize("prec", ["fp32", "ds", "fp64"])
@pytest.mark.parametrize("name", sorted(SYSTEMS))
@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_lists_are_padded_from_elsewhere(name, prec, lanes):
    s = SYSTEMS[name]()
    cfg = mdx.make_config(s.table, prec, 0.002, s.skin, 1, s.n, max_cells=200000, nbr_capacity=80,
                          lanes_per_particle=lanes)
    pool = mdx.MdSystem(cfg)
    pool.attach_system(0, s)
    for steps in (0, 200):
        if steps:
            pool.step(steps)
        ob = pool.observables()[0]
        pos, _, _ = pool.get_state(0)
        f, _ = pool.forces(0)
        ref = O.forces_cells(pos, s.box, s.species, s.table)[0]
        # against the largest force: most particles of a gas carry none (and the
        # pair force is zero at the cutoff, or no pair is near it)
        err = float(np.abs(f - ref).max() / np.abs(ref).max())
        cnt, _ = pool.neighbours(0, cap=1)
        say(f"{name} {prec} lanes {lanes}: lists of {cnt.min()} to {cnt.max()}, {ob['n_rebuilds']} builds, error {err:.2e}")
        assert (cnt % (4 * lanes)).any()
        assert err < TOL_F[prec]
    pool.close()


def test_a_replica_without_a_far_particle_stops():
    """Four particles, each in the lists of the others: nothing to pad with."""
    pos = np.array([[5.0, 5, 5], [6.1, 5, 5], [5, 6.1, 5], [5, 5, 6.1]])
    s = I.System(4, 12.0, pos, np.zeros((4, 3)), np.zeros(4, dtype=np.int32), I.lj_table(2.5), 1.0)
    pool = mdx.MdSystem(mdx.make_config(s.table, "ds", 0.001, 0.3, 1, 4))
    pool.attach_system(0, s)
    pool.step(4)
    with pytest.raises(mdx.MdError):
        pool.observables()
    assert pool.observables(check=False)[0]["status"] & mdx.MD_ST_NO_PAD
    pool.close()
