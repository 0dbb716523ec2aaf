"""dbl_cell_offset1 (the matrix-core list test's positions in FP64), compiled
for the host: the offset that goes with the cell that the sort takes from an
unfolded position.  The folded position's own cell is another one at both ends
of the box."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "md_dev.hpp"
int main()
{
    double x, L;
    int nd;
    while (scanf("%la %la %d", &x, &L, &nd) == 3) {
        const double invL = 1.0 / L;
        const int c = dbl_cell1(x, L, invL, nd);
        double f = x; // the sort's fold
        if (f < 0.0) f += L;
        if (f >= L) f -= L;
        printf("%d %d %a %a\n", c, dbl_cell1(f, L, invL, nd), f, dbl_cell_offset1(x, L, invL, nd));
    }
}
"""


def test_offsets_lie_in_the_cell_of_the_sort(tmp_path):
    src = tmp_path / "offset.cpp"
    src.write_text(SOURCE)
    exe = str(tmp_path / "offset")
    subprocess.run(["hipcc", "--offload-host-only", "-std=c++17", "-O1", "-ffp-contract=off", "-w",
                    "-I" + os.path.join(ROOT, "paper_0912_3824_amd", "csrc"), str(src), "-o", exe], check=True)
    rng = np.random.default_rng(7)
    rows = []
    for L, nd in ((20.155154296590084, 7), (8.4, 3), (31.37, 11), (100.0, 35), (64.0, 22), (9.41e2, 336)):
        eps = np.spacing(L) * np.array([0, 1, 2, 0.26, 0.24, 0.1, 1e-3, 1e-12])
        xs = list(rng.uniform(-0.4, L + 0.4, 400))
        for face in np.concatenate([[0.0, L], rng.integers(1, nd, 20) * L / nd]):
            xs += list(face + eps) + list(face - eps)
        rows += [(float(x), L, nd) for x in xs]
    text = "\n".join(f"{x.hex()} {L.hex()} {nd}" for x, L, nd in rows)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
    out = np.array([float.fromhex(v) if "x" in v else float(v) for v in out]).reshape(-1, 4)
    assert len(out) == len(rows)
    x, L, nd = (np.array(v) for v in zip(*rows))
    cell, again, _, off = out.T
    # the two roundings part at both ends of the box
    assert np.sum((cell == nd - 1) & (again == 0) & (x < 0)) > 10
    assert np.any((cell == nd - 1) & (again == 0) & (x >= L))
    # at most half an edge, to a rounding of x / L times the cells
    assert np.abs(off).max() <= 0.5 + 1e-12
    d = (cell + 0.5 + off) * (L / nd) - x
    d -= L * np.rint(d / L)
    # three roundings of numbers below L
    assert np.all(np.abs(d) <= 4 * np.spacing(L) * 1.0)
