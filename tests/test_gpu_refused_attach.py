"""An attach or a restore that is refused leaves nothing in the arena: what is
attached afterwards, to the same slot or over the same range, runs as in a pool
of its own."""
import time

import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import pool_for
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu

CAP = 96  # list entries: enough at density 0.5 (28 on average), not at 1.4 (129)


def _lj(n, rho, seed):
    return I.make_lj(n, rho=rho, temperature=1.5, jitter=0.05, seed=seed)


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def _faulty(fault, n):
    s = _lj(n, 1.4 if fault == "lists" else 0.5, seed=n)
    if fault == "pos":
        s.pos[n - 1, 2] = np.nan
    elif fault == "vel":
        s.vel[5, 0] = np.inf
    return s, mdx.MD_E_CAPACITY if fault == "lists" else mdx.MD_E_NONFINITE


@pytest.mark.parametrize("fault", ["pos", "vel", "lists"])
@pytest.mark.parametrize("prec", ["ds", "fp64"])
def test_later_replicas_run_as_alone(prec, fault):
    good = {2: _lj(1500, 0.5, 1), 0: _lj(1100, 0.5, 2), 1: _lj(1300, 0.5, 3)}
    bad, status = _faulty(fault, 3000)
    cfg = mdx.make_config(bad.table, prec, 0.002, bad.skin, 3, 6000, nbr_capacity=CAP)
    pool = mdx.MdSystem(cfg)
    pool.attach_system(2, good[2])
    with pytest.raises(mdx.MdError) as e:
        pool.attach_system(0, bad)
    assert e.value.status == status
    pool.attach_system(0, good[0])  # the same slot, fewer particles
    pool.attach_system(1, good[1])  # another slot, over the rest of the range
    pool.step(200)
    assert all(o["n_rebuilds"] > 4 for o in pool.observables())
    for k, s in good.items():
        alone = pool_for([s], prec, dt=0.002, nbr_capacity=CAP)
        alone.step(200)
        assert _same(pool.get_state(k), alone.get_state(0)), k
        alone.close()
    pool.close()


@pytest.mark.parametrize("prec", ["ds", "fp64"])
def test_a_refused_restore_leaves_nothing(prec):
    """A checkpoint whose lists overflow the pool's capacity: the dead slot is
    counted neither by the observables' reduction (its chunks of 4096 particles
    would not fit beside the others') nor by the steps."""
    n = 60000
    dense = _lj(n, 1.4, 4)
    wide = pool_for([dense], prec, dt=0.002)
    blob = wide.save(0)
    wide.close()
    s, t = _lj(n - 5000, 0.5, 5), _lj(1300, 0.5, 6)
    cfg = mdx.make_config(s.table, prec, 0.002, s.skin, 3, n, nbr_capacity=CAP)
    pool = mdx.MdSystem(cfg)
    with pytest.raises(mdx.MdError) as e:
        pool.restore(0, blob, n, dense.box)
    assert e.value.status == mdx.MD_E_CAPACITY
    assert list(pool.poll()[0]) == [-1, -1, -1]
    pool.attach_system(1, s)
    pool.attach_system(0, t)
    pool.step(60)
    obs = pool.observables()
    for k, r in ((1, s), (0, t)):
        alone = pool_for([r], prec, dt=0.002, nbr_capacity=CAP)
        alone.step(60)
        o = alone.observables()[0]
        assert all(np.array_equal(o[q], obs[k][q]) for q in o), k
        assert o["n_rebuilds"] > 1
        assert _same(pool.get_state(k), alone.get_state(0)), k
        alone.close()
    pool.close()


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("prec", ["ds", "fp64"])
def test_input_without_a_finite_position_is_refused_at_once(prec, value):
    """All non-finite positions convert to one cell; a list build of that cell
    (20,000 members in one wave) would take seconds."""
    s = _lj(20000, 0.5, 7)
    cfg = mdx.make_config(s.table, prec, 0.002, s.skin, 1, s.n, nbr_capacity=CAP)
    pool = mdx.MdSystem(cfg)
    pool.attach_system(0, s)
    pool.detach(0)
    t0 = time.perf_counter()
    with pytest.raises(mdx.MdError) as e:
        pool.attach(0, s.n, s.box, s.species, np.full_like(s.pos, value), s.vel)
    assert time.perf_counter() - t0 < 0.5
    assert e.value.status == mdx.MD_E_NONFINITE
    pool.attach_system(0, s)
    pool.step(40)
    alone = pool_for([s], prec, dt=0.002, nbr_capacity=CAP)
    alone.step(40)
    assert _same(pool.get_state(0), alone.get_state(0))
    pool.close()
    alone.close()
