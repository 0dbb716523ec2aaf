"""FP64 positions that the sort takes for the last cell and folds to 0: x so
little below 0 that x + L rounds to L.  On a perfect lattice with a site at 0
the planted particles move there within one step."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import say
from list_order import cells_of, ordered_lists, slots_of
from paper_0912_3824_amd import mdx

pytestmark = pytest.mark.gpu

FORMS = {  # fcc cells per edge, density, cutoff: cells per edge x members per cell
    "product": (12, 0.8442, 2.5),          # 7^3 x 20.2
    "two_items": (8, 1.2, 2.5),            # 4^3 x 32.0
    "candidates": (16, 0.75, I.WCA_RC),    # 19^3 x 2.4
    "members": (39, 0.75, I.WCA_RC),       # 47^3 x 2.3
}


@pytest.mark.parametrize("order", ["row", "hilbert"])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_lists_of_particles_folded_to_zero(form, order):
    n1, rho, rc = FORMS[form]
    n, skin = 4 * n1 ** 3, 0.3
    box = (n / rho) ** (1.0 / 3.0)
    a = box / n1
    g = np.arange(n1)
    unit = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 1, 3)
    basis = np.array([[0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]])
    pos = ((unit + basis) * a).reshape(-1, 3)
    vel = np.where(pos == 0.0, -5e-13, 0.0)  # 5e-16 below 0 after a step; box + that rounds to box
    assert box - 5e-16 == box
    sp, table = np.zeros(n, dtype=np.int32), I.lj_table(rc)
    pool = mdx.MdSystem(mdx.make_config(table, "fp64", 0.001, skin, 1, n, cell_order=order))
    pool.attach(0, n, box, sp, pos, vel)
    pool.step(1)
    pool.rebuild_neighbours()
    now, _, img = pool.get_state(0)
    planted = pos == 0.0
    assert np.all(now[planted] == 0.0) and np.all(img == 0)
    nd = int(np.floor(box / (rc + skin)))
    cells = cells_of(now, box, nd, "fp64")
    cells[planted] = nd - 1  # where the sort counted them
    near = np.nonzero((now < 1.5 * (rc + skin)).any(axis=1) | (now > box - rc - skin).any(axis=1))[0]
    sel = near if len(near) < 4000 else np.sort(np.random.default_rng(1).choice(near, 4000, replace=False))
    ref = ordered_lists(now, box, sp, table, skin, cells, nd, slots_of(pool, 0, n), sel)
    cnt, ids = pool.neighbours(0)
    bad = sum(not np.array_equal(ids[i, :cnt[i]], r) for i, r in zip(sel, ref))
    say(f"box edge, {form} {order}: {planted.any(axis=1).sum()} planted, {bad} of {len(sel)} lists differ")
    assert bad == 0
    pool.close()
