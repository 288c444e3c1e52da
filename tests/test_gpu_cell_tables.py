"""exx_set_cell's device-made tables against the host's: a plan moved to another
cell and back evaluates as the plan it was.  The two sets of tables differ by
rounding alone (FP64: 1e-16 relative a value, amplified in no sum by more than
the 1e-11 that repeated set_cell evaluations are allowed; mixed: values whose
rounding to two BF16 parts falls the other way, 2^-17 relative each)."""
import numpy as np
import pytest
import torch

from paper_2011_07209_amd import exx, synth

from gpu_util import rel1
from test_gpu_cell import _eval, _inputs
from test_gpu_general import CELLS, _cfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("l_max", [0, 5, 6, 8])
def test_set_cell_back_and_forth(l_max, prec):
    h, N = CELLS["triclinic"]
    cfg = _cfg(f"cell-tables-{l_max}", h, N, n_orb=4, R_ME=6.0, l_max=l_max, seed_index=97)
    tol = 1e-11 if prec == "fp64" else 1e-5
    plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, stencil_n=3, cg_tol=cfg.cg_tol,
                    cell_fluctuation=1, precision=exx.EXX_PREC_MIXED if prec == "mixed" else exx.EXX_PREC_FP64)
    try:
        _, _, orb_t, cen_t = _inputs(cfg)
        E0, S0, D0 = _eval(plan, orb_t, cen_t)[:3]
        h0 = np.asarray(cfg.h)
        plan.set_cell(h0 * 1.01)
        E1 = _eval(plan, orb_t, cen_t)[0]
        plan.set_cell(h0)
        E2, S2, D2 = _eval(plan, orb_t, cen_t)[:3]
    finally:
        plan.close()
    assert rel1(E1, E0) > 1e-4
    assert rel1(E2, E0) <= tol and rel1(S2, S0) <= tol and rel1(D2, D0) <= tol
