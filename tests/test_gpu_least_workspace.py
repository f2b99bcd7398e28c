"""Solvers in the least workspace that mg_create takes (levels kept as boxes):
the solution of the full one to the solves' own tolerance, through
set_coefficients, and a workspace between the two sizes."""

import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import lib, rel_l2, to_global
from test_gpu_nodal import _nodal_mf

CASES = [
    # cfg maker, opts
    (lambda: W.config_lognormal(64, 32), {}),
    (lambda: W.config_lognormal(64, 16), dict(precision=1, tune=2)),
    (lambda: W.config_lognormal(64, 32), dict(krylov=1, aggregate=1)),
    (lambda: W.config_lognormal(64, 32), dict(krylov=1, precision=1)),
    (W.config_c0, dict(min_bottom_edge=8)),  # singular; a bottom of 4096 cells
    (lambda: W.config_lognormal(72, 72), dict(min_bottom_edge=18)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("make,opts", CASES)
def test_least_workspace_solves(make, opts):
    P = lib()
    cfg = make()
    print(f"[least workspace] {cfg['n']}^3 {opts}", flush=True)
    n, boxes, per = cfg["n"], cfg["boxes"], cfg["periodic"]
    f = cfg["rhs"] - (cfg["rhs"].mean() if all(per) else 0.0)
    rhs = P.MultiFab.from_numpy(boxes, W.scatter_cells(f, boxes), 0)

    def faces(scale):
        if cfg.get("faces") is None:
            return None
        return [P.MultiFab.from_numpy(boxes, W.scatter_faces(scale * cfg["faces"][d], boxes, d), 0,
                                      ixtype=tuple(int(e == d) for e in range(3)))
                for d in range(3)]

    out = []
    for least in (False, True):
        s = P.MLMG(boxes, W.domain_box(n), per, cfg["alpha"], cfg["beta"], b=faces(1.0),
                   opts=dict(dict(tune=0), **opts), least_workspace=least)
        size = s.workspace.numel()
        sol = []
        for scale in (1.0, 3.0):
            if scale != 1.0:
                s.set_coefficients(b=faces(scale))
            phi = s.cell_mf(1, fill=0.0)
            info = s.solve(phi, rhs, 1e-11)
            torch.cuda.synchronize()
            assert info["converged"]
            sol.append(to_global(phi, boxes, n))
        s.close()
        out.append((size, sol))
    assert out[1][0] < out[0][0]
    for x, y in zip(out[0][1], out[1][1]):
        assert rel_l2(y, x) <= 1e-8  # two residual tolerances times the condition, as elsewhere


@pytest.mark.gpu
def test_between_the_sizes_and_composite(monkeypatch):
    """One byte short of the full size works as the least does, bit for bit where
    the bottom has no column layout; and the composite solver."""
    print("[least workspace] between the sizes, composite", flush=True)
    P = lib()
    import paper_2009_12009_amd.solver as S
    cfg = W.config_lognormal(64, 32)
    n, boxes = cfg["n"], cfg["boxes"]
    rhs = P.MultiFab.from_numpy(boxes, W.scatter_cells(cfg["rhs"], boxes), 0)
    size_of = S.workspace_bytes
    out = []
    for least in (False, True):
        if not least:
            monkeypatch.setattr(S, "workspace_bytes", lambda *a: size_of(*a) - 257)
        s = P.MLMG(boxes, W.domain_box(n), (False,) * 3, cfg["alpha"], cfg["beta"],
                   opts=dict(tune=0), least_workspace=least)
        monkeypatch.setattr(S, "workspace_bytes", size_of)
        phi = s.cell_mf(1, fill=0.0)
        s.solve(phi, rhs, 1e-10)
        torch.cuda.synchronize()
        out.append(to_global(phi, boxes, n))
        s.close()
    assert np.array_equal(out[0], out[1])

    fine = [((16, 16, 16), (47, 47, 47))]
    sol = []
    for least in (False, True):
        s = P.CompositeMLMG([W.domain_box(32)], fine, W.domain_box(32), 0.0, 1.0,
                            opts=dict(tune=0), least_workspace=least)
        rng = np.random.default_rng(1)
        pc, rc = P.MultiFab(s.boxes, 1, fill=0.0), P.MultiFab.from_numpy(
            s.boxes, [rng.uniform(-1, 1, (32, 32, 32))], 0)
        pf, rf = P.MultiFab(s.fine_boxes, 1, fill=0.0), P.MultiFab.from_numpy(
            s.fine_boxes, [rng.uniform(-1, 1, (32, 32, 32))], 0)
        info = s.solve(pc, pf, rc, rf, 1e-11)
        torch.cuda.synchronize()
        assert info["converged"]
        sol.append(np.concatenate([pc.valid_numpy()[0].ravel(), pf.valid_numpy()[0].ravel()]))
        s.close()
    assert rel_l2(sol[1], sol[0]) <= 1e-8


# bytes mg_nodal_create took before the tail's plan and the sweeps' dot products
# had a place in the workspace
NODAL = [
    (64, 32, (True, False, True), {}, 19984128),
    (24, 12, (True, True, True), dict(krylov=1), 1902080),
    (40, 40, (False, False, False), {}, 4865568),
    (128, 64, (False, False, False), {}, 148303872),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,edge,per,opts,size", NODAL)
def test_nodal_in_its_former_workspace(n, edge, per, opts, size, monkeypatch):
    print(f"[least workspace] nodal {n} {per} {opts}", flush=True)
    P = lib()
    import paper_2009_12009_amd.nodal as N
    boxes = W.uniform_boxes(n, edge)
    rng = np.random.default_rng(6)
    f = rng.standard_normal(W.nodal_unknown_shape(n, per))
    f -= f.mean()
    sol = []
    for former in (False, True):
        if former:
            monkeypatch.setattr(N, "nodal_workspace_bytes", lambda *a: size)
        s = P.NodalMLMG(boxes, W.domain_box(n), per, opts=dict(tune=0, **opts))
        phi = s.node_mf(0, fill=0.0)
        info = s.solve(phi, _nodal_mf(P, boxes, f, n, per, 0), 1e-10)
        torch.cuda.synchronize()
        assert info["converged"]
        sol.append(np.concatenate([x.ravel() for x in phi.to_numpy()]))
        s.close()
    assert rel_l2(sol[1], sol[0]) <= 1e-8
    monkeypatch.setattr(N, "nodal_workspace_bytes", lambda *a: size - 4096)
    with pytest.raises(P.MGError) as e:
        P.NodalMLMG(boxes, W.domain_box(n), per, opts=dict(tune=0, **opts))
    assert e.value.code == P._lib.MG_ERR_WORKSPACE
