"""Which small spheres take the preconditioned CG: on the last size below the
line of each kind of plan the iteration counts are the plain CG's (solve_depth =
1), on the first size above it they are far fewer (27 of 55 at the smallest), and
both sides agree with the plain CG within the parity bars."""
import numpy as np
import pytest

from paper_2011_07209_amd import exx, synth

from gpu_util import gpu_eval
from test_gpu_general import CELLS, _cfg
from test_gpu_precond import _check

pytestmark = pytest.mark.gpu

LINES = [("ortho", "fp64", 1, 7), ("ortho", "fp64", 3, 7), ("ortho", "mixed", 1, 7), ("ortho", "mixed", 2, 6),
         ("ortho", "mixed", 3, 5), ("hexagonal", "fp64", 1, 6), ("hexagonal", "fp64", 3, 6), ("hexagonal", "mixed", 3, 5),
         ("triclinic", "fp64", 2, 6), ("triclinic", "mixed", 1, 7), ("triclinic", "mixed", 2, 6)]


@pytest.mark.parametrize("cell,prec,n,line", LINES)
def test_line_of_small_spheres(cell, prec, n, line):
    p = exx.EXX_PREC_MIXED if prec == "mixed" else exx.EXX_PREC_FP64
    for m in (line - 1, line, 1):   # points from the centre to the surface along the narrowest axis
        kw = dict(n_orb=6, R_pair=7.0, l_max=4, stencil_n=n, cg_tol=1e-10, seed_index=60 + m)
        if cell == "ortho":
            R = 0.24 * (m + 0.05)
            cfg = synth.custom(key=f"small-{n}-{m}", cell=(12.0, 11.5, 12.0), grid=(50, 50, 55), R_PE=R, R_ME=R + 1.5, **kw)
        else:
            h, N = CELLS[cell]
            hi = np.linalg.inv(np.asarray(h))
            # the longest grid step along an axis reaches past m points exactly when the sphere does:
            # its extent on axis a is R |row a of h^-1| N_a points
            R = (m + 0.05) / min(np.linalg.norm(hi[a]) * N[a] for a in range(3))
            cfg = _cfg(f"small-{cell}-{n}-{m}", h, N, R_PE=R, R_ME=R + 2.0, **kw)
        orbs = synth.make_orbitals(cfg)
        phi = synth.fill_orbitals(cfg, orbs)
        g, o = gpu_eval(cfg, orbs, phi, precision=p), gpu_eval(cfg, orbs, phi, precision=p, solve_depth=1)
        a, b = g["stats"]["cg_iter_sum"], o["stats"]["cg_iter_sum"]
        print(f"[small {cell} {prec} n {n}] points {m} line {line}: iterations {a} plain {b}", flush=True)
        assert a < 0.75 * b if m >= line else abs(a - b) <= 0.02 * b + g["stats"]["n_pairs"]
        _check(g, o, prec, cfg.n_orb)
