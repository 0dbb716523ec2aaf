"""The order of the list entries (own cell, then opposite cell pairs; A before B
members, in slot order) in every form of the list build, entry by entry: which
form a replica gets depends on its cells, their members and how many replicas
rebuild together, and a trajectory's bits depend on the order."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import near_cutoff, say
from list_order import cells_of, ordered_lists, slots_of
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu


def _droplet(n, rho, mean, rc):
    """A ball of fcc lattice in an empty box of mean density `mean`."""
    box, a = (n / mean) ** (1.0 / 3.0), (4.0 / rho) ** (1.0 / 3.0)
    m = int(np.ceil(box / a))
    full = I.fcc_positions(4 * m ** 3, m * a, None)
    full = full[(full < box - 0.5).all(axis=1)]
    pos = full[np.argsort(((full - box / 2) ** 2).sum(axis=1), kind="stable")[:n]]
    rng = np.random.default_rng(n)
    pos = np.mod(pos + rng.uniform(-0.05, 0.05, pos.shape), box)
    vel = rng.normal(size=pos.shape)
    return I.System(n, box, pos, vel - vel.mean(axis=0), np.zeros(n, dtype=np.int32), I.lj_table(rc), 1.0)


FORMS = {
    # one replica rebuilds with fine shares, eight together with whole products
    "single": lambda: I.make_ka(601, 0.7, jitter=0.06, seed=1),                            # one cell
    "mixture": lambda: I.make_ka(1500, 0.7, jitter=0.06, seed=2),                          # 3^3 x 55.6
    "mixture_4": lambda: I.make_ka(2905, 0.7, jitter=0.06, seed=3),                        # 4^3 x 45.4
    "product": lambda: I.make_lj(10007, rho=0.75, jitter=0.09, seed=4),                    # 8^3 x 19.5
    "candidates": lambda: I.make_lj(3001, rho=0.75, jitter=0.09, rc=I.WCA_RC, seed=5),     # 11^3 x 2.3
    "long_lists": lambda: I.make_lj(5003, rho=1.2, jitter=0.09, rc=2.8, seed=6),           # 5^3 x 40, lists of 150
    "wide": lambda: I.make_lj(4001, rho=0.8442, jitter=0.09, rc=4.5, seed=7),              # 3^3 x 148, lists of 390
    "droplet": lambda: _droplet(6000, 0.9, 0.15, 2.5),                                     # 12^3 x 3.5, some of 20
    "members": lambda: I.make_lj(240000, rho=0.75, jitter=0.09, rc=I.WCA_RC, seed=8),      # 48^3 x 2.2
    "wide_large": lambda: I.make_lj(60000, rho=0.8442, jitter=0.09, rc=4.5, seed=9),       # 8^3 x 117
}


@pytest.mark.parametrize("prec", ["ds", "fp64"])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_entries_are_in_order(form, prec):
    s = FORMS[form]()
    n = s.n
    copies = 8 if n < 20000 else 1
    order = "hilbert" if form in ("mixture_4", "droplet") else "row"
    cfg = mdx.make_config(s.table, prec, s.dt, s.skin, copies, copies * n, cell_order=order, max_cells=400000,
                          max_density=1.2)
    rl = float(max(s.table.rcut[a, b] for a in range(2) for b in range(2))) + s.skin
    nd = int(np.floor(s.box / rl))
    nd = nd if nd >= 3 else 1
    pool = mdx.MdSystem(cfg)
    pool.attach_system(0, s)
    pos, _, _ = pool.get_state(0)
    sel = np.arange(n) if n < 5000 else np.sort(np.random.default_rng(3).choice(n, 1500, replace=False))
    if n < 100000:
        near = near_cutoff(pos, s.box, s.species, s.table, lambda a, b: s.table.rcut[a, b] + s.skin)
        sel = sel[~near[sel]]
    cells = cells_of(pos, s.box, nd, prec)
    ref = None
    for what in ("attached", "rebuilt alone", "rebuilt together"):
        if what == "rebuilt together":
            if copies == 1:
                break
            for k in range(1, copies):
                pool.attach_system(k, s)
        if what != "attached":
            pool.rebuild_neighbours()
        slots = slots_of(pool, 0, n)
        if ref is None:
            first = slots
            ref = ordered_lists(pos, s.box, s.species, s.table, s.skin, cells, nd, slots, sel)
        assert np.array_equal(slots, first)
        for k in {0, copies - 1} if what == "rebuilt together" else {0}:
            cnt, ids = pool.neighbours(k, cap=640)
            bad = sum(not np.array_equal(ids[i, :cnt[i]], r) for i, r in zip(sel, ref))
            say(f"list order, {form} {prec} {what}: lists of {cnt.min()} to {cnt.max()}, {bad} of {len(sel)} differ")
            assert bad == 0
    pool.close()


@pytest.mark.parametrize("prec", ["ds", "fp64"])
@pytest.mark.parametrize("count", [32, 33, 96, 97])
def test_many_single_cell_replicas(count, prec):
    """How many members share an item goes by how many replicas rebuild together;
    sizes of one member, of less and of more than a wave, at odd places."""
    sizes = [601, 1, 31, 64, 65, 2, 187]
    box = 8.0  # two cells of 2.8 an edge
    reps = []
    for k, n in enumerate(sizes):
        rng = np.random.default_rng(k)
        pos = I.fcc_positions(n, box, rng, 0.05)
        reps.append(I.System(n, box, pos, rng.normal(size=(n, 3)), I.species_80_20(n, rng), I.ka_table(), 0.7))
    cfg = mdx.make_config(reps[0].table, prec, 0.001, 0.3, count, 601 * count)
    pool = mdx.MdSystem(cfg)
    for k in range(count):
        pool.attach_system(k, reps[k % len(reps)])
    pool.rebuild_neighbours()
    for k in list(range(7)) + [count - 1]:
        s = reps[k % len(reps)]
        pos, _, _ = pool.get_state(k)
        slots = slots_of(pool, k, s.n)
        ref = ordered_lists(pos, box, s.species, s.table, 0.3, None, 1, slots, np.arange(s.n))
        near = near_cutoff(pos, box, s.species, s.table, lambda a, b: s.table.rcut[a, b] + 0.3)
        cnt, ids = pool.neighbours(k, cap=200)
        bad = [i for i in range(s.n) if not near[i] and not np.array_equal(ids[i, :cnt[i]], ref[i])]
        say(f"{count} single cells {prec}, replica of {s.n}: lists of {cnt.min()} to {cnt.max()}, {len(bad)} differ")
        assert not bad
    pool.close()


def test_a_replica_of_heavy_cells_comes_and_goes():
    """The list build's form follows the replicas attached, also in captured
    graphs, and changes no bit of the others' trajectories."""
    light = I.make_lj(3001, rho=0.4, temperature=1.5, jitter=0.05, rc=4.0, seed=11)  # 4^3 x 46.9
    heavy = I.make_lj(4001, rho=0.8442, temperature=1.5, jitter=0.05, rc=4.0, seed=12)  # 3^3 x 148
    for slots in (1, 2):
        cfg = mdx.make_config(light.table, "ds", 0.002, light.skin, slots, 8000)
        pool = mdx.MdSystem(cfg)
        alone = mdx.md_init([light], "ds", dt=0.002)
        beside = mdx.md_init([heavy], "ds", dt=0.002)
        pool.attach_system(0, light)
        for k in range(3):
            if slots == 1 and k == 1:  # through the heavy replica and back, by a checkpoint
                blob = pool.save(0)
                pool.detach(0)
                pool.attach_system(0, heavy)
                pool.step(64)
                beside.step(64)
                assert all(np.array_equal(x, y) for x, y in zip(pool.get_state(0), beside.get_state(0)))
                pool.detach(0)
                pool.restore(0, blob, light.n, light.box)
            if slots == 2 and k == 1:
                pool.attach_system(1, heavy)
            if slots == 2 and k == 2:
                beside.step(64)
                assert all(np.array_equal(x, y) for x, y in zip(pool.get_state(1), beside.get_state(0)))
                pool.detach(1)
            pool.step(64)
            alone.step(64)
            assert all(np.array_equal(x, y) for x, y in zip(pool.get_state(0), alone.get_state(0))), (slots, k)
        assert alone.observables()[0]["n_rebuilds"] > 3
        for p in (pool, alone, beside):
            p.close()
