"""A plan goes on unchanged after a refused exx_eval_noalloc: exx_eval keeps
the plan's solver (as many CG iterations as a plan that was never refused, and
the same energy to the last bit: the per-pair work is the same), and the same
call is refused again."""
import pytest
import torch

from paper_2011_07209_amd import exx

from test_zz_no_alloc import DEV, _inputs

pytestmark = pytest.mark.gpu


def _eval(plan, orb_t, cen_t):
    E = torch.zeros(1, dtype=torch.float64, device=DEV)
    plan.eval(orb_t, cen_t, E)
    torch.cuda.synchronize()
    st = plan.stats()
    return E.item(), st["cg_iter_sum"], st["n_pairs"], st["solve_threads"], st["solve_depth"]


@pytest.mark.parametrize("autotune", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_evaluations_after_a_refusal(precision, autotune):
    cfg, orb_t, cen_t = _inputs(4)
    # more pairs than the scratch array holds
    opt = dict(stencil_n=cfg.stencil_n, cg_tol=cfg.cg_tol, max_pairs=4_000_000, autotune=autotune,
               precision=exx.EXX_PREC_MIXED if precision == "mixed" else exx.EXX_PREC_FP64)
    args = (cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max)
    ref_plan = exx.Plan(*args, **{**opt, "autotune": 0})
    plain_plan = exx.Plan(*args, **{**opt, "autotune": 0, "solve_depth": 1})
    plan = exx.Plan(*args, **opt)
    try:
        ref, plain = _eval(ref_plan, orb_t, cen_t), _eval(plain_plan, orb_t, cen_t)
        assert ref[1] < 0.5 * plain[1]
        for _ in range(2):
            with pytest.raises(exx.ExxError) as e:
                plan.eval(orb_t, cen_t, noalloc=True)
            assert e.value.status == exx.EXX_EINVAL
            got = _eval(plan, orb_t, cen_t)
            print(f"[after a refusal, {precision} autotune {autotune}] E, iterations, pairs, threads, depth: {got} "
                  f"never refused {ref} plain {plain}", flush=True)
            assert got[2] == ref[2] and abs(got[0] - ref[0]) <= 1e-9 * abs(ref[0])
            assert got[1] < 0.5 * plain[1]
            if not autotune:
                assert got == ref
    finally:
        for p in (plan, ref_plan, plain_plan):
            p.close()
