"""The default workgroup of the preconditioned CG on wide spheres: 512 threads for
FP64 orthorhombic classes of 2,049 to 3,072 columns (six each), 1024 on both
sides of them and for general cells and mixed plans in single columns.  Against
the plain CG within the parity bars."""
import numpy as np
import pytest

from paper_2011_07209_amd import exx, synth

from gpu_util import gpu_eval
from test_gpu_general import _cell, _cfg
from test_gpu_precond import _check

pytestmark = pytest.mark.gpu


# points from the centre to the surface: 25.4 (2,025 columns), 25.8 (2,085), 31.0 (3,001), 31.6 (3,133)
@pytest.mark.parametrize("cell,prec,points,threads", [
    ("ortho", "fp64", 25.4, 1024), ("ortho", "fp64", 25.8, 512), ("ortho", "fp64", 31.0, 512),
    ("ortho", "fp64", 31.6, 1024), ("ortho", "mixed", 31.6, 1024), ("triclinic", "fp64", 29.0, 1024),
    ("triclinic", "fp64", 33.0, 1024)])
def test_default_threads(cell, prec, points, threads):
    kw = dict(n_orb=2, R_pair=8.0, l_max=4, stencil_n=3, cg_tol=1e-11, seed_index=89)
    if cell == "ortho":
        R = points * 0.16
        cfg = synth.custom(key=f"threads-{points}", cell=(15.36, 15.36, 15.36), grid=(96, 96, 96), R_PE=R, R_ME=R + 0.8, **kw)
        cols = sum(x * x + y * y <= points * points for x in range(-40, 41) for y in range(-40, 41))
        assert (2048 < cols <= 3072) == (threads == 512)
    else:
        h = _cell(14.4, 14.4, 14.4, 80, 95, 100)
        R = points * 0.15
        cfg = _cfg(f"threads-tri-{points}", np.asarray(h), (96, 96, 96), R_PE=R, R_ME=R + 1.2, **kw)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    opt = dict(precision=exx.EXX_PREC_MIXED if prec == "mixed" else exx.EXX_PREC_FP64, cg_layout=1)
    g, o = gpu_eval(cfg, orbs, phi, **opt), gpu_eval(cfg, orbs, phi, solve_depth=1, **opt)
    print(f"[threads {cell} {prec} {points}] {g['stats']['solve_threads']} iterations {g['stats']['cg_iter_sum']} plain "
          f"{o['stats']['cg_iter_sum']}", flush=True)
    assert g["stats"]["solve_threads"] == threads
    assert g["stats"]["cg_iter_sum"] < 0.5 * o["stats"]["cg_iter_sum"]
    _check(g, o, prec, cfg.n_orb)
