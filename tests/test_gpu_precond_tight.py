"""Solves that take their residual down to the rounding of the first one: cg_tol
near and below the FP64 epsilon (the residual that the stop test reads is the
recursion's), and mixed plans whose update threshold lets the FP32 recursion run
on towards the FP32 epsilon.  The plan keeps the preconditioned CG only where
its coarse residuals stay accurate; on both sides of that line it does what the
plain CG of the same plan does (solve_depth = 1), with its energy within the
parity bar of a solve to 1e-12."""
import dataclasses

import pytest

from paper_2011_07209_amd import exx, synth

from gpu_util import gpu_eval, rel1
from test_gpu_parity import MIXED_E_PER_MOLECULE, TOL_D, TOL_E, TOL_S
from test_gpu_precond import _config

pytestmark = pytest.mark.gpu

CASES = [("ortho", 1), ("ortho", 3), ("hexagonal", 3), ("triclinic", 3)]


@pytest.mark.parametrize("tol", [1e-14, 0.99e-14, 1e-16, 1e-18])
@pytest.mark.parametrize("cell,n", CASES)
def test_tolerances_below_the_epsilon(cell, n, tol):
    cfg = _config(cell, n, 3.9)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    ref = gpu_eval(cfg, orbs, phi)
    cfg = dataclasses.replace(cfg, cg_tol=tol)
    g, p = gpu_eval(cfg, orbs, phi), gpu_eval(cfg, orbs, phi, solve_depth=1)
    print(f"[{cfg.key} tol {tol:g}] iterations {g['stats']['cg_iter_sum']} plain {p['stats']['cg_iter_sum']} "
          f"residual {g['stats']['max_rel_residual']:.2e} E {g['E']:.15g} {ref['E']:.15g}", flush=True)
    assert p["stats"]["n_unconverged"] == 0 and g["stats"]["n_unconverged"] == 0
    assert g["stats"]["max_rel_residual"] <= tol
    assert (g["stats"]["cg_iter_sum"] < 0.5 * p["stats"]["cg_iter_sum"]) == (tol >= 1e-14)
    assert rel1(g["E"], ref["E"]) <= TOL_E
    assert rel1(g["sigma"], ref["sigma"]) <= TOL_S and rel1(g["D"], ref["D"]) <= TOL_D


@pytest.mark.parametrize("delta,tol", [(1e-4, 1e-10), (1e-6, 1e-10), (0.99e-6, 1e-10), (1e-8, 1e-6), (1e-8, 1e-7)])
@pytest.mark.parametrize("cell,n", CASES)
def test_update_thresholds_towards_the_fp32_epsilon(cell, n, delta, tol):
    cfg = dataclasses.replace(_config(cell, n, 3.9), cg_tol=tol)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    kw = dict(want_D=False, precision=exx.EXX_PREC_MIXED, refine_delta=delta)
    g, p = gpu_eval(cfg, orbs, phi, **kw), gpu_eval(cfg, orbs, phi, solve_depth=1, **kw)
    o = gpu_eval(dataclasses.replace(cfg, cg_tol=1e-12), orbs, phi)
    st, sp = g["stats"], p["stats"]
    print(f"[{cfg.key} delta {delta:g} tol {tol:g}] iterations {st['cg_iter_sum']} plain {sp['cg_iter_sum']} updates "
          f"{st['refine_passes_max']} unconverged {st['n_unconverged']} {sp['n_unconverged']} E {g['E']:.12f} "
          f"{p['E']:.12f} {o['E']:.12f}", flush=True)
    assert st["cg_restarts"] == 0 and st["n_unconverged"] <= sp["n_unconverged"]
    assert (st["cg_iter_sum"] < 0.5 * sp["cg_iter_sum"]) == (max(delta, tol) >= 1e-6)
    if max(delta, tol) < 1e-6:
        assert g["E"] == p["E"]
    # (a solve to a tolerance above 1e-7 leaves an error of that order; where the
    # plain CG stops at the cap, there is no converged energy to compare with)
    if sp["n_unconverged"] == 0:
        assert abs(g["E"] - o["E"]) <= (MIXED_E_PER_MOLECULE + 10 * tol) * cfg.n_orb / 4
