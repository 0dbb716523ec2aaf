"""The sums of a correlation pass (species split, ragged last workgroup, the
fewest and the most lags) against the oracle's scheme on the frames read back
at the samples.  In FP64 both see the same numbers up to the rounding of the
unwrapped positions (1e-15 of the box against displacements above 1e-3) and of
the sums (n eps), well below the tolerance of 1e-9."""
import math

import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import pool_for, say
from oracle import tcf as OT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels,block", [(257, 2, 2), (500, 1, 33), (1023, 2, 3), (4097, 1, 10)])
def test_pass_sums(n, levels, block):
    s = I.make_ka(n, 1.0, jitter=0.05, seed=n)
    q = 2 * math.pi * 6 / s.box
    pool = pool_for([s], "fp64")
    t = pool.tcf(0, levels, block, q=q)
    ref = OT.Blocking(levels, block, s.species, q)
    for m in range(block + 4):
        if m:
            pool.step(4)
        pos, vel, img = pool.get_state(0)
        t.sample()
        ref.sample(pos + img * s.box, vel)
    lags, vals, terms = t.read()
    rl, rv, rt = ref.result()
    assert np.array_equal(terms, rt) and np.array_equal(lags, rl)
    ok = rt > 0
    err = np.abs(vals[ok] - rv[ok]) / np.abs(rv[ok])
    say(f"n {n} block {block}: largest relative difference {err.max():.2g}")
    assert err.max() < 1e-9
    pool.close()
