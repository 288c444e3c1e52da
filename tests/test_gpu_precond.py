"""The preconditioned CG against the plain CG of the same plan options (chosen
by solve_depth = 1) and, through it, the FP64 oracle's bars: both solve to
||r|| <= tol ||b||, so E, sigma and D agree within the parity tests' bars and
the preconditioned iteration count is less than half the plain one.

The cases are the edges of its dispatch: stencil half-widths, the window form
with stored and recomputed A p, arms leaving the sweep plane, padded columns,
one to eight columns per thread, spheres of a few points (coarsest grids of one
point or none), and previous solutions as starts."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2011_07209_amd import exx, synth

from gpu_util import gpu_eval, rel1
from test_gpu_general import CELLS, _cfg
from test_gpu_parity import MIXED_D, MIXED_E_PER_MOLECULE, MIXED_S, TOL_D, TOL_E, TOL_S

pytestmark = pytest.mark.gpu


def _config(cell, n, R):
    kw = dict(n_orb=4, R_pair=7.0, R_PE=R, R_ME=R + 1.2, l_max=5, stencil_n=n, cg_tol=1e-12, seed_index=80 + n)
    if cell == "ortho":
        return synth.custom(key=f"pc-ortho-{n}-{R}", cell=(11.0, 12.0, 10.5), grid=(50, 56, 46), **kw)
    h, N = CELLS[cell]
    return _cfg(f"pc-{cell}-{n}-{R}", h, N, **kw)


def _check(a, b, prec, n_orb):
    assert a["stats"]["n_unconverged"] == 0 and b["stats"]["n_unconverged"] == 0
    assert [tuple(x) for x in a["pairs"]["ij"]] == [tuple(x) for x in b["pairs"]["ij"]]
    if prec == "fp64":
        assert rel1(a["E"], b["E"]) <= TOL_E
        assert rel1(a["sigma"], b["sigma"]) <= TOL_S and rel1(a["D"], b["D"]) <= TOL_D
    else:
        assert abs(a["E"] - b["E"]) <= MIXED_E_PER_MOLECULE * n_orb / 4
        assert rel1(a["sigma"], b["sigma"]) <= MIXED_S and rel1(a["D"], b["D"]) <= MIXED_D


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cell,n,R,threads", [
    ("ortho", 1, 3.9, 0), ("ortho", 2, 3.9, 1024), ("ortho", 3, 3.9, 0), ("ortho", 3, 3.9, 512),
    ("ortho", 3, 0.7, 0), ("ortho", 1, 1.5, 1024), ("ortho", 3, 2.2, 512),
    ("hexagonal", 3, 4.0, 0), ("monoclinic", 2, 4.0, 512),
    ("triclinic", 3, 4.0, 0), ("rhombohedral", 1, 3.0, 1024), ("triclinic", 2, 4.0, 512)])
def test_preconditioned_matches_plain(cell, n, R, threads, prec):
    cfg = _config(cell, n, R)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    p = exx.EXX_PREC_MIXED if prec == "mixed" else exx.EXX_PREC_FP64
    g = gpu_eval(cfg, orbs, phi, precision=p, solve_threads=threads)
    o = gpu_eval(cfg, orbs, phi, precision=p, solve_threads=threads, solve_depth=1)
    print(f"[{cfg.key} {prec} {threads}] iterations {g['stats']['cg_iter_sum']} plain {o['stats']['cg_iter_sum']} "
          f"threads {g['stats']['solve_threads']}", flush=True)
    _check(g, o, prec, cfg.n_orb)
    if R >= 2.0:
        assert g["stats"]["cg_iter_sum"] < 0.5 * o["stats"]["cg_iter_sum"]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_wide_sphere_columns_per_thread(prec):
    """More than six columns per thread of a 512-thread workgroup."""
    cfg = synth.custom(key="pc-wide", cell=(15.0, 15.0, 15.0), grid=(96, 96, 96), n_orb=2, R_pair=8.0, R_PE=5.2,
                       R_ME=6.0, l_max=4, stencil_n=3, cg_tol=1e-12, seed_index=88)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    p = exx.EXX_PREC_MIXED if prec == "mixed" else exx.EXX_PREC_FP64
    runs = [gpu_eval(cfg, orbs, phi, precision=p, solve_threads=t) for t in (512, 1024)]
    assert [r["stats"]["solve_threads"] for r in runs] == [512, 1024]
    assert abs(runs[0]["stats"]["cg_iter_sum"] - runs[1]["stats"]["cg_iter_sum"]) <= 0.1 * runs[1]["stats"]["cg_iter_sum"]
    _check(runs[0], gpu_eval(cfg, orbs, phi, precision=p, solve_depth=1), prec, cfg.n_orb)
    _check(runs[0], runs[1], prec, cfg.n_orb)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_an_iteration_cap_of_plain_cg_runs_plain_cg(prec):
    """A cap below what the plain CG needs is one of plain CG steps."""
    cfg = _config("ortho", 3, 3.9)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    p = exx.EXX_PREC_MIXED if prec == "mixed" else exx.EXX_PREC_FP64
    orb_t = torch.from_numpy(phi).to("cuda:0")
    cen_t = torch.from_numpy(np.ascontiguousarray(orbs.centres)).to("cuda:0")
    plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, stencil_n=3, cg_tol=1e-12,
                    cg_max_iter=40, precision=p)
    try:
        E = torch.zeros(1, dtype=torch.float64, device="cuda:0")
        plan.eval(orb_t, cen_t, E, None, None)
        torch.cuda.synchronize()
        st = plan.stats(allow_noconv=True)
        assert st["n_unconverged"] == st["n_pairs"] and st["cg_iter_max"] == 40
    finally:
        plan.close()
