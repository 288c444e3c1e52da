"""exx_set_cell while an evaluation of the plan's old cell is still in flight on
the null stream and the plan is bound to another (non-blocking) stream: the
evaluation reads the old cell's tables to its end, so its energy is the one of
an undisturbed evaluation to the last bit (sums in a fixed order)."""
import numpy as np
import pytest
import torch

from paper_2011_07209_amd import exx

from test_gpu_cell import _inputs
from test_gpu_general import CELLS, _cfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("how", ["enqueued", "graph"])
def test_set_cell_waits_for_the_null_stream(how, prec):
    h, N = CELLS["triclinic"]
    cfg = _cfg("cell-order", h, N, n_orb=4, R_ME=6.0, l_max=6, seed_index=98)
    plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, stencil_n=3, cg_tol=cfg.cg_tol,
                    cell_fluctuation=1, max_pairs=32,
                    precision=exx.EXX_PREC_MIXED if prec == "mixed" else exx.EXX_PREC_FP64)
    try:
        _, _, orb_t, cen_t = _inputs(cfg)
        E = torch.zeros(1, dtype=torch.float64, device=orb_t.device)
        plan.eval(orb_t, cen_t, E)
        torch.cuda.synchronize()
        assert plan.stats()["n_pairs"] > 0
        want = E.item()
        side = torch.cuda.Stream()
        g = None
        if how == "graph":
            g = torch.cuda.CUDAGraph()
            with torch.cuda.stream(side):
                plan.set_stream(side)
                with torch.cuda.graph(g, stream=side):
                    plan.eval(orb_t, cen_t, E)
        # work in front of the evaluation, so that it starts after the call below
        a = torch.randn(4096, 4096, device=orb_t.device)
        b = torch.empty_like(a)
        for _ in range(40):
            torch.mm(a, a, out=b)
        torch.cuda.synchronize()
        E.zero_()
        for _ in range(40):
            torch.mm(a, a, out=b)
        if g is None:
            plan.eval(orb_t, cen_t, E)
        else:
            g.replay()
        plan.set_stream(side)
        plan.set_cell(1.02 * np.asarray(cfg.h))
        torch.cuda.synchronize()
        got = E.item()
        plan.eval(orb_t, cen_t, E)
        torch.cuda.synchronize()
        print(f"[cell order {how} {prec}] E={got:.15g} undisturbed {want:.15g} next cell {E.item():.15g}", flush=True)
        assert got == want
        assert abs(E.item() - want) > 1e-4 * abs(want)
        del g
    finally:
        plan.close()
