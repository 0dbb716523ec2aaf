"""Every form of the list build (chosen by cells and members per cell) against
the oracle's neighbour sets, at the sizes where a form's edges lie: few
members per cell (one lane per candidate; one lane per member above 100,000
cells), cells of more than 32 members (two items per cell), lists longer than
the build's buffer, and neighbourhoods beyond its chunk table."""
import numpy as np
import pytest

import md_inputs as I
from gpu_helpers import near_cutoff, pool_for, say
from oracle import oracle as O
from oracle.upload import state_after_upload

pytestmark = pytest.mark.gpu

FORMS = {
    # n, density, cutoff, skin: cells per edge x members per cell
    "candidates": (3001, 0.75, I.WCA_RC, 0.3),       # 11^3 x 2.3
    "members": (240000, 0.75, I.WCA_RC, 0.3),        # 48^3 x 2.2
    "product": (10007, 0.75, 2.5, 0.3),              # 8^3 x 19.5
    "two_items": (2905, 1.2, 2.5, 0.3),              # 4^3 x 45.4
    "long_lists": (5003, 1.2, 2.8, 0.3),             # 5^3 x 40.0, lists of 150
    "beyond_table": (4001, 0.8442, 4.5, 0.5),        # 3^3 x 148
}


@pytest.mark.parametrize("prec", ["ds", "fp64"])
@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_lists_match_oracle(prec, form, lanes):
    n, rho, rc, skin = FORMS[form]
    if n > 100000 and (lanes != 2):
        pytest.skip("one lane count at the large size")
    s = I.make_lj(n, rho=rho, jitter=0.09, rc=rc, skin=skin, seed=n)
    pool = pool_for([s], prec, lanes_per_particle=lanes)
    pos, _, _ = state_after_upload(s.pos, s.vel, s.box, prec)
    sel = np.arange(n) if n <= 20000 else np.sort(np.random.default_rng(3).choice(n, 400, replace=False))
    ref = O.neighbours(pos, s.box, s.species, s.table, s.skin, sel=sel.astype(np.int32))
    near = near_cutoff(pos, s.box, s.species, s.table, lambda a, b: rc + skin, band=1e-6) if n <= 20000 else None
    for again in (False, True):
        if again:  # the same through the sort
            pool.rebuild_neighbours()
        cnt, ids = pool.neighbours(0, cap=1024)
        bad = 0
        for k, i in enumerate(sel):
            same = np.array_equal(np.sort(ids[i, :cnt[i]]), ref[k])
            if not same and not (near is not None and near[i]):
                bad += 1
        say(f"{form} {prec} lanes {lanes}: mean list {cnt.mean():.1f}, {bad} lists differ")
        assert bad == 0
    pool.close()
