"""GPU parity of the nodal kernels where their form changes: rows that end one
node past a wavefront, on it and before it, walls and wraps at those ends, levels
of one plane per work-group and of many.  Against the oracle."""

import numpy as np
import pytest
import torch

import oracle.nodal as ON
import workloads as W
from gpu_util import lib
from test_gpu_nodal import _gpu, _inputs, _nodal_mf, _solve_pair, _unknowns

F, T = False, True


@pytest.mark.gpu
@pytest.mark.parametrize("n,per", [(66, (F, F, F)), (64, (T, F, F)), (64, (F, F, F)),
                                   (66, (T, T, F)), (130, (F, T, T)), (130, (F, F, F)),
                                   (12, (T, F, T))])
def test_apply(n, per):
    print(f"[nodal shapes] apply {n} {per}", flush=True)
    P = lib()
    boxes = [W.domain_box(n)]
    sigma, _ = _inputs(n, boxes, per)
    s = _gpu(n, boxes, per, sigma, dict(min_bottom_edge=3))
    x = np.random.default_rng(3).standard_normal(W.nodal_unknown_shape(n, per))
    phi = _nodal_mf(P, boxes, x, n, per, 0)
    out = s.node_mf(0, fill=np.nan)
    s.apply(phi, out)
    torch.cuda.synchronize()
    got, _ = _unknowns(out, boxes, n, per)
    ref = ON.apply_nodal(ON.make_nodal_level(sigma, per), x)
    # 27 terms of rounding each
    assert np.abs(got - ref).max() <= 1e-13 * np.abs(ref).max()
    s.close()


# extents of the levels' unknowns: 71, 35, 17, bottom 8; 55, 27, 13, bottom 6;
# 64, 32, 16, 8, bottom 4 with wraps; 39, 19, 9, bottom 4; bottom 11 (more nodes
# than one work-group's lanes)
CYCLES = [
    (72, (F, F, F), 4, {}),
    (56, (F, F, F), 4, {}),
    (64, (T, F, T), 4, {}),
    (40, (F, F, T), 4, dict(use_graph=0)),
    (48, (F, F, F), 12, {}),
    (24, (T, T, T), 3, {}),
    (40, (F, T, F), 4, dict(nu1=1, nu2=3)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,per,mbe,opts", CYCLES)
def test_cycles(n, per, mbe, opts):
    """Residual before every cycle as the oracle's to 1e-6, solution of three
    cycles to rounding."""
    print(f"[nodal shapes] cycles {n} {per} {opts}", flush=True)
    boxes = W.uniform_boxes(n, n // 2)
    nu = {k: v for k, v in opts.items() if k.startswith("nu")}
    sigma, f = _inputs(n, boxes, per)
    info, got, _, _, _ = _solve_pair(n, boxes, per, mbe, max_iter=3, tol=1e-14, opts=opts)
    ophi, oinfo = ON.nodal_solve(sigma, per, f, 1e-14, opts=ON.NodalOpts(
        bottom_tol=1e-12, min_bottom_cells=mbe, max_iter=3, **nu))
    h, o = np.array(info["history"]), np.array(oinfo["history"])
    assert np.all(np.abs(h - o) <= 1e-6 * o)
    # three cycles of rounding and the bottoms' 1e-12
    assert np.abs(got - ophi).max() <= 1e-10 * np.abs(ophi).max()


@pytest.mark.gpu
@pytest.mark.parametrize("n,per", [(64, (F, F, F)), (66, (F, T, F)), (48, (T, T, T))])
def test_krylov_same_solution(n, per):
    """Conjugate gradients reach the V-cycles' solution: both residuals are below
    1e-11 max|f|, the smallest eigenvalue of A is above 1 over the unit cube (more
    than pi^2 times the smallest coefficient)."""
    boxes = [W.domain_box(n)]
    a = _solve_pair(n, boxes, per, 4, tol=1e-11, opts=dict(max_iter=300))
    b = _solve_pair(n, boxes, per, 4, tol=1e-11, opts=dict(max_iter=300, krylov=1))
    assert a[0]["converged"] and b[0]["converged"]
    _, f = _inputs(n, boxes, per)
    # 2-norms: |r|_2 <= sqrt(N) max|r|
    bound = 2e-11 * np.abs(f).max() * np.sqrt(f.size)
    assert np.linalg.norm(a[1] - b[1]) <= bound
