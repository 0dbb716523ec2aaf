"""Small pools of one slot sum a list in four lanes (terms a quarter each, one
component to a lane); pools of two slots in one.  Trajectories, forces,
energies and observables keep the same bits: every precision, one and two
lists a particle, plain, mixed-cutoff and smoothed pairs, lists from a few
entries to many rows, one cell and many."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import say
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu

SYSTEMS = {
    "gas": lambda: I.make_lj(301, rho=0.05, jitter=0.2, rc=2.5, skin=0.3, seed=5),
    "one_cell": lambda: I.make_ka(500, 0.7, seed=6),
    "mixture": lambda: I.make_ka(1999, 0.7, seed=7),
    "fluid": lambda: I.make_lj(5003, rho=0.8442, jitter=0.08, rc=2.5, skin=0.3, seed=8),
    "smooth": lambda: I.smoothed(I.make_lj(1201, rho=0.7, jitter=0.08, rc=2.5, skin=0.3, seed=9), 0.005),
}


def run(s, prec, lanes, slots):
    cfg = mdx.make_config(s.table, prec, 0.002, s.skin, slots, s.n, lanes_per_particle=lanes, max_cells=4096)
    pool = mdx.MdSystem(cfg)
    pool.attach_system(0, s)
    out = []
    for steps in (1, 50):
        pool.step(steps)
        f, e = pool.forces(0)
        out += [np.asarray(f).copy(), np.asarray(e).copy()]
        out += [x.copy() for x in pool.get_state(0)]
        o = pool.observables()[0]
        out.append(np.array([float(v) for _, v in sorted(o.items()) if np.isscalar(v)]))
    pool.close()
    return out


@pytest.mark.parametrize("prec", ["fp32", "ds", "mixed64", "fp64"])
@pytest.mark.parametrize("lanes", [1, 2])
@pytest.mark.parametrize("name", sorted(SYSTEMS))
def test_quads_keep_the_bits(name, lanes, prec):
    s = SYSTEMS[name]()
    a, b = run(s, prec, lanes, 1), run(s, prec, lanes, 2)
    say(f"{name} {prec} lanes {lanes}: largest force {np.abs(a[0]).max():.3g}")
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert np.isfinite(x.astype(float)).all() and np.array_equal(x, y)
