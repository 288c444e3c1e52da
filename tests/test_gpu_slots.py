"""A plan whose persistent workgroups' CG vectors exceed the device's memory
(asked for by solve_groups, between what the plain and the preconditioned CG's
would take): the evaluation runs with fewer workgroups and gives what the
default number gives, to the last bit (each pair is solved by one workgroup)."""
import pytest
import torch

from paper_2011_07209_amd import exx, synth

from test_gpu_precond import _config

pytestmark = pytest.mark.gpu


def test_more_workgroups_than_memory():
    cfg = _config("ortho", 3, 3.9)
    orbs = synth.make_orbitals(cfg)
    dev = torch.device("cuda:0")
    orb_t = torch.from_numpy(synth.fill_orbitals(cfg, orbs)).to(dev)
    cen_t = torch.from_numpy(orbs.centres).to(dev)

    def run(**kw):
        plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, stencil_n=3, cg_tol=cfg.cg_tol,
                        **kw)
        try:
            n_pe = plan.geometry()["n_pe"]
            E = torch.zeros(1, dtype=torch.float64, device=dev)
            S = torch.zeros(9, dtype=torch.float64, device=dev)
            plan.eval(orb_t, cen_t, E, None, S)
            torch.cuda.synchronize()
            st = plan.stats()
            return E.item(), S.cpu(), st["cg_iter_sum"], n_pe
        finally:
            plan.close()

    ref = run()
    free, _ = torch.cuda.mem_get_info()
    # bytes a point and slot: 16 plain, more than 48 preconditioned
    groups = int(free / (32 * ref[3]))
    got = run(solve_groups=groups)
    print(f"[slots] groups {groups} E {got[0]:.15g} {ref[0]:.15g} iterations {got[2]}", flush=True)
    assert got[0] == ref[0] and torch.equal(got[1], ref[1]) and got[2] == ref[2]
