"""The conversion and the sort of an attached replica (done on the device):
slot order by (species, cell, id), positions of any image, refused inputs."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import pool_for
from oracle.upload import state_after_upload
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["row", "hilbert"])
@pytest.mark.parametrize("prec", ["fp32", "ds", "mixed64", "fp64"])
@pytest.mark.parametrize("n", [500, 3001, 20161, 20165])  # 20164 x 52 bytes fill the staging buffer
def test_order_and_images(prec, n, order):
    s = I.make_ka(n, 0.7, jitter=0.06, seed=n)
    rng = np.random.default_rng(n)
    shift = rng.integers(-3, 4, size=(n, 3))
    far = s.pos + shift * s.box
    cfg = mdx.make_config(s.table, prec, s.dt, s.skin, 3, 2 * n + 900, cell_order=order)
    pool = mdx.MdSystem(cfg)
    other = I.make_ka(800, 0.6, jitter=0.06, seed=3)
    pool.attach_system(2, other)
    pool.attach(0, n, s.box, s.species, far, s.vel)
    pos, vel, img = pool.get_state(0)
    rpos, rvel, rimg = state_after_upload(far, s.vel, s.box, prec)
    assert np.array_equal(pos, rpos) and np.array_equal(vel, rvel) and np.array_equal(img, rimg)
    blob = pool.save(0)
    ids = np.frombuffer(blob, np.int32)[-4 * n:].reshape(n, 4)[:, 3]
    assert np.array_equal(np.sort(ids), np.arange(n))
    nd = int(np.floor(s.box / (2.5 + s.skin)))
    nd = nd if nd >= 3 else 1
    if prec == "fp64":
        cell = np.minimum((pos * (1.0 / s.box) * nd).astype(int), nd - 1)
    else:
        cell = ((np.rint(pos * (2.0 ** 32 / s.box)).astype(np.uint64) % 2 ** 32) * nd >> np.uint64(32)).astype(int)
    rank = mdx.cell_order_ranks(nd, order)[cell[:, 0] + nd * (cell[:, 1] + nd * cell[:, 2])]
    assert np.array_equal(ids, np.lexsort((np.arange(n), rank, s.species)))
    # the same replica once more, in another slot: the same run
    pool.attach(1, n, s.box, s.species, far, s.vel)
    pool.step(30)
    a, b = pool.get_state(0), pool.get_state(1)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    pool.close()


@pytest.mark.parametrize("n", [700, 30000])
def test_refused_inputs_leave_the_slot_free(n):
    s = I.make_ka(n, 0.7, jitter=0.06, seed=8)
    cfg = mdx.make_config(s.table, "ds", s.dt, s.skin, 2, n + 100)
    pool = mdx.MdSystem(cfg)
    bad = s.pos.copy()
    bad[n - 1, 2] = np.nan
    inf = s.vel.copy()
    inf[5, 0] = np.inf
    sp = s.species.copy()
    sp[n // 2] = 2
    for args, status in (((s.species, bad, s.vel), mdx.MD_E_NONFINITE), ((s.species, s.pos, inf), mdx.MD_E_NONFINITE),
                         ((sp, s.pos, s.vel), -1), ((sp, bad, s.vel), mdx.MD_E_NONFINITE)):
        with pytest.raises(mdx.MdError) as e:
            pool.attach(0, n, s.box, *args)
        assert e.value.status == status
    pool.attach_system(0, s)
    with pytest.raises(mdx.MdError) as e:  # no room: a fault of the input goes first
        pool.attach(1, n, s.box, s.species, bad, s.vel)
    assert e.value.status == mdx.MD_E_NONFINITE
    with pytest.raises(mdx.MdError) as e:
        pool.attach(1, n, s.box, s.species, s.pos, s.vel)
    assert e.value.status == mdx.MD_E_CAPACITY
    pool.step(20)
    alone = pool_for([s], "ds")
    alone.step(20)
    assert all(np.array_equal(x, y) for x, y in zip(pool.get_state(0), alone.get_state(0)))
    pool.close()
    alone.close()
