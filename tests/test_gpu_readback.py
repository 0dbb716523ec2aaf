"""Frames and forces read back by particle id against the checkpoint's own
words, on both sides of the size up to which a read-back is staged."""
import ctypes

import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import pool_for

pytestmark = pytest.mark.gpu

NW = {"fp32": 2, "ds": 3, "mixed64": 3, "fp64": 3}
STAGED = 17476  # largest replica whose 60 bytes a particle fit 1 MiB


def decode(blob, n, prec, box):
    """Positions, velocities and images by id from a checkpoint's state words
    (and its meta words, the last 16 n bytes)."""
    head = len(blob) - 16 * n * (NW[prec] + 2 * (2 if prec == "fp64" else 1) + 1)
    w = np.frombuffer(blob, np.uint8)[head:head + 16 * n * NW[prec]].reshape(NW[prec], n, 16)
    if prec == "fp32":
        f = w.copy().view(np.float32)
        x, v = f[0, :, :3].astype(np.float64), f[1, :, :3].astype(np.float64)
    elif prec == "ds":
        f = w.copy().view(np.float32).astype(np.float64)
        x = np.stack([f[0, :, 0] + f[0, :, 3], f[0, :, 1] + f[1, :, 0], f[0, :, 2] + f[1, :, 1]], 1)
        v = np.stack([f[1, :, 2] + f[2, :, 1], f[1, :, 3] + f[2, :, 2], f[2, :, 0] + f[2, :, 3]], 1)
    else:
        f = w.copy().view(np.float64)
        x = np.stack([f[0, :, 0], f[0, :, 1], f[1, :, 0]], 1)
        v = np.stack([f[1, :, 1], f[2, :, 0], f[2, :, 1]], 1)
    meta = np.frombuffer(blob, np.int32)[-4 * n:].reshape(n, 4)
    s = np.floor(x / box)
    q = x - s * box
    img = meta[:, :3] + s.astype(np.int32)
    img = img + (q >= box) - (q < 0)
    q = np.where(q >= box, q - box, q)
    q = np.where(q < 0, q + box, q)
    order = np.argsort(meta[:, 3])
    return q[order], v[order], img[order]


@pytest.mark.parametrize("prec", sorted(NW))
@pytest.mark.parametrize("n", [501, STAGED, STAGED + 1, 30001])
def test_frames_equal_the_checkpoint(prec, n):
    s = I.make_ka(n, 0.7, jitter=0.06, seed=n)
    small = I.make_ka(777, 0.6, jitter=0.06, seed=5)
    pool = pool_for([small, s], prec)  # the replica does not start at slot 0 of the arena
    pool.step(40)
    pos, vel, img = pool.get_state(1)
    ref = decode(pool.save(1), n, prec, s.box)
    assert np.array_equal(pos, ref[0]) and np.array_equal(vel, ref[1]) and np.array_equal(img, ref[2])
    # outputs the caller does not ask for
    v2 = np.zeros((n, 3))
    st = pool.lib.md_get_state(pool.h, 1, None, v2.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), None)
    assert st == 0 and np.array_equal(v2, vel)
    assert pool.lib.md_get_state(pool.h, 1, None, None, None) == 0
    # forces and energies together and alone
    f, e = pool.forces(1)
    e2 = np.zeros(n)
    st = pool.lib.md_forces(pool.h, 1, None, e2.ctypes.data_as(ctypes.POINTER(ctypes.c_double)))
    assert st == 0 and np.array_equal(e, e2)
    assert abs(f.sum(axis=0)).max() < 1e-2 * np.abs(f).max() and np.isfinite(f).all()
    o = pool.observables()[1]
    assert abs(e.sum() - o["epot"]) <= 1e-12 * abs(o["epot"])
    # reading changes nothing
    again = pool.get_state(1)
    assert all(np.array_equal(a, b) for a, b in zip(again, (pos, vel, img)))
    pool.close()
