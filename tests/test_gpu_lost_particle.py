"""A replica that stops because its sort lost a particle (one that crossed more
than a cell in a step) can still be read: the state is that of the step, for
every particle, also where frames and thermostat draws went through the sort's
scratch arrays before."""
import numpy as np
import pytest

import md_inputs as I
from oracle.upload import state_after_upload
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "ds", "mixed64", "fp64"])
@pytest.mark.parametrize("n,slots", [(3001, 1), (30000, 1), (30000, 2)])
def test_state_of_a_stopped_replica(prec, n, slots):
    s = I.make_ka(n, 0.7, jitter=0.06, seed=8)
    pool = mdx.MdSystem(mdx.make_config(s.table, prec, s.dt, s.skin, slots, slots * n))
    if slots > 1:
        pool.attach_system(1, I.make_ka(2000, 0.7, jitter=0.06, seed=9))
    pool.attach_system(0, s)
    pool.step(60)  # fills the scratch arrays
    pool.thermostat(0, 0.7, 3, 0)
    pool.get_state(0)
    pool.detach(0)
    k, vel = n // 3, s.vel.copy()
    vel[k] = [9000.0, 0.0, 0.0]  # 9 in a step: three cells
    pool.attach(0, n, s.box, s.species, s.pos, vel)
    pool.get_state(0)
    pool.thermostat(0, 0.7, 3, 1)
    pool.detach(0)
    pool.attach(0, n, s.box, s.species, s.pos, vel)
    pool.step(3)
    steps, status = pool.poll()
    assert steps[0] == 1 and status[0] & mdx.MD_ST_LOST
    pos, v, img = pool.get_state(0)
    p0, v0, img0 = state_after_upload(s.pos, vel, s.box, prec)
    # one step from the input: dt v, and dt^2 F with |F| below 1e4 on the jittered lattice
    d = pos + (img - img0) * s.box - (p0 + s.dt * v0)
    assert np.abs(d).max() < 1e-2
    assert np.abs(v - v0).max() < 20.0 and np.all(np.abs(pos - s.box / 2) <= s.box / 2)
    pool.close()
