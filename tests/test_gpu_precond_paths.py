"""Branches of the preconditioned CG that an ordinary evaluation does not take:
previous solutions as starts, launches that several sphere classes share (beside
classes that run the plain CG), the iteration cap and the mixed solve's restarts."""
import numpy as np
import pytest
import torch

from paper_2011_07209_amd import exx, synth

from gpu_util import gpu_eval, rel1
from test_gpu_general import CELLS, _cfg
from test_gpu_parity import MIXED_D, MIXED_E_PER_MOLECULE, MIXED_S, TOL_D, TOL_E, TOL_S
from test_gpu_precond import _config

pytestmark = pytest.mark.gpu

PREC = {"fp64": exx.EXX_PREC_FP64, "mixed": exx.EXX_PREC_MIXED}
DEV = torch.device("cuda:0")


def _two_steps(cfg, prec, **kw):
    """E, sigma, D and statistics of the second of two steps, its orbitals displaced by up to a grid step."""
    plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, stencil_n=cfg.stencil_n, cg_tol=cfg.cg_tol,
                    precision=PREC[prec], max_pairs=64, **kw)
    try:
        orbs = synth.make_orbitals(cfg)
        E = torch.zeros(1, dtype=torch.float64, device=DEV)
        S = torch.zeros(9, dtype=torch.float64, device=DEV)
        for step in range(2):
            orb_t = torch.from_numpy(synth.fill_orbitals(cfg, orbs)).to(DEV)
            cen_t = torch.from_numpy(np.ascontiguousarray(orbs.centres)).to(DEV)
            D = torch.empty_like(orb_t)
            plan.eval(orb_t, cen_t, E, D, S)
            torch.cuda.synchronize()
            orbs = synth.displace(cfg, orbs, 1, amplitude=0.03)
        return E.item(), S.cpu().numpy(), D.cpu().numpy(), plan.stats(allow_noconv=True)
    finally:
        plan.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cell,n", [("ortho", 3), ("ortho", 1), ("hexagonal", 2), ("triclinic", 3), ("rhombohedral", 3)])
def test_warm_starts(cell, n, prec):
    cfg = _config(cell, n, 3.9)
    warm, plain, cold = (_two_steps(cfg, prec, warm_start=1), _two_steps(cfg, prec, warm_start=1, solve_depth=1),
                         _two_steps(cfg, prec))
    print(f"[warm {cell} {n} {prec}] iterations {warm[3]['cg_iter_sum']} plain {plain[3]['cg_iter_sum']} cold "
          f"{cold[3]['cg_iter_sum']} warm pairs {warm[3]['warm_pairs']}", flush=True)
    assert warm[3]["n_unconverged"] == 0 and plain[3]["n_unconverged"] == 0
    assert warm[3]["warm_pairs"] == plain[3]["warm_pairs"] > 0
    assert warm[3]["cg_iter_sum"] < min(0.5 * plain[3]["cg_iter_sum"], cold[3]["cg_iter_sum"])
    for other in (plain, cold):
        if prec == "fp64":
            assert rel1(warm[0], other[0]) <= TOL_E and rel1(warm[1], other[1]) <= TOL_S
            assert rel1(warm[2], other[2]) <= TOL_D
        else:
            assert abs(warm[0] - other[0]) <= MIXED_E_PER_MOLECULE * cfg.n_orb / 4
            assert rel1(warm[1], other[1]) <= MIXED_S and rel1(warm[2], other[2]) <= MIXED_D


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cell", ["ortho", "triclinic"])
def test_classes_that_share_a_launch(cell, prec):
    """Seven radii: the two smallest run the plain CG, the others the preconditioned
    one, several to a launch.  Each pair gives what a plan of its radius alone
    gives: a right-hand side whose moments are summed in other chunks (their number
    follows the classes), solved to the same tolerance in as many iterations, one
    more or less."""
    classes = (1.0, 0.55, 7)
    kw = dict(n_orb=14, R_pair=6.0, R_PE=4.3, R_ME=6.4, l_max=4, stencil_n=3, cg_tol=1e-11, seed_index=87)
    if cell == "ortho":
        cfg = synth.custom(key="share-ortho", cell=(13.0, 12.0, 12.5), grid=(56, 52, 54), R_PE_classes=classes,
                           R_orb_range=(1.0, 4.3), **kw)
    else:
        h, N = CELLS[cell]
        cfg = _cfg("share-tri", h, N, R_PE_classes=classes, R_orb_range=(1.0, 4.3), **kw)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    g, o = gpu_eval(cfg, orbs, phi, precision=PREC[prec]), gpu_eval(cfg, orbs, phi, precision=PREC[prec], solve_depth=1)
    st = g["stats"]
    print(f"[classes {cell} {prec}] pairs {st['class_pairs']} threads {st['class_threads']} iterations {st['cg_iter_sum']} "
          f"plain {o['stats']['cg_iter_sum']}", flush=True)
    assert st["n_unconverged"] == 0 and sum(1 for p in st["class_pairs"] if p) >= 5
    if prec == "fp64":
        assert rel1(g["E"], o["E"]) <= TOL_E and rel1(g["sigma"], o["sigma"]) <= TOL_S and rel1(g["D"], o["D"]) <= TOL_D
    else:
        assert abs(g["E"] - o["E"]) <= MIXED_E_PER_MOLECULE * cfg.n_orb / 4
        assert rel1(g["sigma"], o["sigma"]) <= MIXED_S and rel1(g["D"], o["D"]) <= MIXED_D
    ij = g["pairs"]["ij"]
    mean = 0.5 * (orbs.R_orb[ij[:, 0]] + orbs.R_orb[ij[:, 1]])
    cls = np.clip(np.floor((mean - classes[0]) / classes[1] + 0.5), 0, classes[2] - 1).astype(int)
    assert [int((cls == k).sum()) for k in range(classes[2])] == st["class_pairs"]
    one = dict(stencil_n=3, cg_tol=cfg.cg_tol, precision=PREC[prec])
    orb_t, cen_t = torch.from_numpy(phi).to(DEV), torch.from_numpy(np.ascontiguousarray(orbs.centres)).to(DEV)
    for k in np.unique(cls):
        plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, classes[0] + k * classes[1], cfg.R_ME, cfg.l_max,
                        solve_threads=st["class_threads"][k], **one)
        try:
            plan.eval(orb_t, cen_t)
            torch.cuda.synchronize()
            r = plan.pair_results()
        finally:
            plan.close()
        at = np.flatnonzero(cls == k)
        assert np.array_equal(r["ij"], ij) and np.abs(r["iters"][at] - g["pairs"]["iters"][at]).max() <= 1
        assert np.abs(r["E"][at] - g["pairs"]["E"][at]).max() <= (TOL_E if prec == "fp64" else MIXED_E_PER_MOLECULE)


@pytest.mark.parametrize("cell,n", [("ortho", 3), ("hexagonal", 3), ("triclinic", 3), ("ortho", 1)])
def test_iteration_cap(cell, n):
    """A mixed plan with a tolerance below what its FP64 residual can reach runs to
    the cap of the preconditioned CG, and keeps the solution it has."""
    cfg = _config(cell, n, 3.9)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    cap = 8 * (2 * 25 + 1)
    o = gpu_eval(cfg, orbs, phi, precision=exx.EXX_PREC_MIXED)
    kw = dict(stencil_n=n, cg_tol=1e-20, precision=exx.EXX_PREC_MIXED, cg_max_iter=cap)
    plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, **kw)
    try:
        E = torch.zeros(1, dtype=torch.float64, device=DEV)
        plan.eval(torch.from_numpy(phi).to(DEV), torch.from_numpy(np.ascontiguousarray(orbs.centres)).to(DEV), E)
        torch.cuda.synchronize()
        st = plan.stats(allow_noconv=True)
        res = plan.pair_results()
    finally:
        plan.close()
    print(f"[cap {cell} {n}] iterations {st['cg_iter_sum']} residual {st['max_rel_residual']:.2e} updates "
          f"{st['refine_passes_max']} E {E.item():.12f} {o['E']:.12f}", flush=True)
    assert st["status"] == exx.EXX_ENOCONV and st["n_cg_cap"] == st["n_pairs"] == st["n_unconverged"] > 0
    assert np.all(res["iters"] == cap) and np.all(res["exit"] == exx.EXX_CG_CAP) and np.all(res["restarts"] == 0)
    assert st["max_rel_residual"] <= 1e-12
    assert abs(E.item() - o["E"]) <= MIXED_E_PER_MOLECULE * cfg.n_orb / 4


@pytest.mark.parametrize("n", [1, 3])
def test_iteration_cap_fp64(n):
    """A grid five times coarser along the sweep, where the preconditioned CG takes
    more iterations than the smallest cap that it accepts: FP64 solves stop there
    with the solution of that many steps (its residual is reported)."""
    cfg = synth.custom(key=f"cap64-{n}", cell=(11.0, 11.0, 10.5), grid=(110, 110, 21), n_orb=2, R_pair=7.0, R_PE=3.6,
                       R_ME=3.8 + 0.5 * n, l_max=4, stencil_n=n, cg_tol=1e-14, seed_index=3)
    orbs = synth.make_orbitals(cfg)
    phi = synth.fill_orbitals(cfg, orbs)
    cap = 8 * (2 * 7 + 1)
    o, p = gpu_eval(cfg, orbs, phi), gpu_eval(cfg, orbs, phi, cg_max_iter=cap - 1)
    g = gpu_eval(cfg, orbs, phi, cg_max_iter=cap)
    st, res = g["stats"], g["pairs"]
    print(f"[cap fp64 {n}] iterations {st['cg_iter_sum']} of {o['stats']['cg_iter_sum']} residual "
          f"{st['max_rel_residual']:.2e} plain {p['stats']['max_rel_residual']:.2e} E {g['E']:.12f} {o['E']:.12f}", flush=True)
    assert o["stats"]["n_unconverged"] == 0 and st["n_cg_cap"] == st["n_pairs"] == st["n_unconverged"] > 0
    assert np.all(res["iters"] == cap) and np.all(res["exit"] == exx.EXX_CG_CAP)
    assert p["stats"]["cg_iter_max"] == cap - 1   # one less: that many steps of the plain CG
    assert 1e-14 < st["max_rel_residual"] <= 1e-9 and st["max_rel_residual"] < 1e-2 * p["stats"]["max_rel_residual"]
    assert rel1(g["E"], o["E"]) <= 10 * TOL_E


@pytest.mark.parametrize("depth", [0, 1])
def test_restarts_end(depth):
    """Grid steps whose Laplacian is too large for FP32: every sweep of the FP32
    recursion gives a norm that is not finite, each solve restarts three times
    and reports that, with both solvers."""
    s = 1e-21
    cfg = synth.custom(key="restart", cell=(11.0 * s, 12.0 * s, 10.5 * s), grid=(50, 56, 46), n_orb=3, R_pair=7.0 * s,
                       R_PE=3.0 * s, R_ME=4.2 * s, l_max=2, stencil_n=3, cg_tol=1e-10, seed_index=83)
    rng = np.random.default_rng(5)
    orb_t = torch.from_numpy(rng.standard_normal((3, 46, 56, 50))).to(DEV)
    cen_t = torch.from_numpy(rng.uniform(0.0, 10.0 * s, (3, 3))).to(DEV)
    plan = exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, stencil_n=3, cg_tol=1e-10,
                    precision=exx.EXX_PREC_MIXED, solve_depth=depth)
    try:
        plan.eval(orb_t, cen_t)
        torch.cuda.synchronize()
        st = plan.stats(allow_noconv=True)
        res = plan.pair_results()
    finally:
        plan.close()
    print(f"[restarts depth {depth}] pairs {st['n_pairs']} exits {res['exit'].tolist()} restarts {res['restarts'].tolist()} "
          f"iterations {res['iters'].tolist()}", flush=True)
    assert st["n_unconverged"] == st["n_pairs"] > 0
    assert np.all(res["restarts"] == 3)
    assert np.all((res["exit"] == exx.EXX_CG_BREAKDOWN) | (res["exit"] == exx.EXX_CG_NONFINITE))
