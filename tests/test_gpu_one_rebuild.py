"""Pools of one slot sort and build their lists in one launch up to 49,152
particles, all others in two: the same replica in a pool of one slot and in
one of two slots keeps the same bits through captured steps, eager ones and
forced rebuilds (sizes: one cell, one sort unit, remainders, the rule's edge
and beyond it)."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import say
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu

CASES = [(130, "ds"), (601, "fp32"), (1003, "mixed64"), (4000, "fp64"), (10007, "ds"), (30001, "fp64"),
         (49152, "fp32"), (49153, "ds")]


def run(s, prec, slots):
    cfg = mdx.make_config(s.table, prec, 0.002, s.skin, slots, s.n, lanes_per_particle=2)
    pool = mdx.MdSystem(cfg)
    pool.attach_system(0, s)
    out = []
    for steps in (1, 70, 33):
        pool.step(steps)
        out += [x.copy() for x in pool.get_state(0)]
        pool.rebuild_neighbours()
        pool.rebuild_neighbours()
        out += [x.copy() for x in pool.neighbours(0, cap=512)]
    o = pool.observables()[0]
    pool.close()
    return out, o["n_rebuilds"], o["status"]


@pytest.mark.parametrize("n,prec", CASES)
def test_one_launch_keeps_the_bits(n, prec):
    s = I.make_lj(n, rho=0.8, jitter=0.08, rc=2.5, skin=0.2, seed=n)
    (a, na, sa), (b, nb, sb) = run(s, prec, 1), run(s, prec, 2)
    say(f"n {n} {prec}: {na} rebuilds")
    assert sa == sb == 0 and na == nb and na >= 7
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
