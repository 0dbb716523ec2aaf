"""The order of a Verlet list's entries, computed on the host (test
infrastructure): the own cell, then each half-space offset o followed by -o,
and within a cell the A members, then the B members, in slot order."""
import numpy as np

from gpu_helpers import pair_distances


def slots_of(pool, slot, n):
    """Slot order of a replica's particles: slots[id]."""
    ids = np.frombuffer(pool.save(slot), np.int32)[-4 * n:].reshape(n, 4)[:, 3]
    out = np.empty(n, dtype=int)
    out[ids] = np.arange(n)
    return out


def cells_of(pos, box, nd, prec):
    """Cell coordinates of positions in [0, box), as the mode bins them."""
    if prec == "fp64":
        return np.minimum((pos * (1.0 / box) * nd).astype(int), nd - 1)
    x = np.rint(pos * (2.0 ** 32 / box)).astype(np.uint64) % 2 ** 32
    return (x * np.uint64(nd) >> np.uint64(32)).astype(int)


def visits():
    """visit[dz + 1, dy + 1, dx + 1]: when the cell at an offset is visited."""
    v = np.zeros((3, 3, 3), dtype=int)
    half = [(z, y, x) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1) if (z, y, x) > (0, 0, 0)]
    for k, (z, y, x) in enumerate(half):
        v[z + 1, y + 1, x + 1] = 2 * k + 1
        v[1 - z, 1 - y, 1 - x] = 2 * k + 2
    return v


def ordered_lists(pos, box, species, table, skin, cells, nd, slots, sel):
    """Neighbour ids of the particles `sel`, each in list order (nd = 1: one
    cell; the order is then that of the slots)."""
    rl = np.array([[table.rcut[a, b] + skin for b in range(2)] for a in range(2)])
    sp = species if table.n_species > 1 else np.zeros(len(pos), dtype=int)
    i, j, r = pair_distances(pos, box, float(rl.max()))
    keep = (r < rl[sp[i], sp[j]]) & np.isin(i, sel)
    i, j = i[keep], j[keep]
    v = np.zeros(len(i), dtype=int)
    if nd > 1:
        o = (cells[j] - cells[i] + 1) % nd  # 0, 1, 2
        assert o.max() <= 2
        v = visits()[o[:, 2], o[:, 1], o[:, 0]]
    at = np.lexsort((slots[j], sp[j], v, i))
    i, j = i[at], j[at]
    first, last = np.searchsorted(i, sel), np.searchsorted(i, sel, side="right")
    return [j[a:b] for a, b in zip(first, last)]
