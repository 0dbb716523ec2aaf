"""A pool of one slot sorts and builds its lists in one launch or in two, by the
cells of its replica and how often time step and skin let it rebuild: replicas
on either side of the rule come and go in one pool, through captured graphs, and
run as in a pool of two slots, which always takes two launches."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import say
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu

# time step, skin, and the sizes at density 0.75: cells per edge 4 .. 14; with
# 0.001 and 0.3 every size takes one launch, with 0.002 and 0.25 only those of up
# to 1,380 cells
CASES = [("fp32", 0.001, 0.3, (2000, 49152, 10007)), ("ds", 0.002, 0.25, (2000, 49152, 22000, 30001)),
         ("mixed64", 0.002, 0.25, (30001, 22000)), ("fp64", 0.001, 0.3, (49000, 1003))]


def _run(pool, s, steps):
    pool.attach_system(0, s)
    out = []
    for k in steps:
        pool.step(k)
        out += [x.copy() for x in pool.get_state(0)]
    pool.rebuild_neighbours()
    out += [x.copy() for x in pool.neighbours(0)]
    o = pool.observables()[0]
    pool.detach(0)
    return out, o


@pytest.mark.parametrize("prec,dt,skin,sizes", CASES)
def test_either_form_keeps_the_bits(prec, dt, skin, sizes):
    table = I.lj_table(2.5)
    pools = [mdx.MdSystem(mdx.make_config(table, prec, dt, skin, slots, 49152)) for slots in (1, 2)]
    for n in sizes:
        s = I.make_lj(n, rho=0.75, jitter=0.08, skin=skin, seed=n)
        (a, oa), (b, ob) = (_run(p, s, (1, 64, 33)) for p in pools)
        say(f"rebuild rule, {prec} dt {dt} n {n}: {oa['n_rebuilds']} rebuilds")
        assert oa["status"] == ob["status"] == 0 and oa["n_rebuilds"] == ob["n_rebuilds"] >= 4
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
    for p in pools:
        p.close()
