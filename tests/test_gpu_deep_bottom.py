"""GPU parity of solves whose CG bottom is preconditioned by its own
coarsenings: bottoms just above the size where that begins, odd extents along
walls and periodic directions on one and on several levels, a hierarchy whose
last levels fit the one-work-group tail and one where they do not, a tolerance
that the preconditioned iterations do not reach.

Tolerance: the operator is an M-matrix with row sums of at least alpha * min a,
so a residual of at most tol * max|f| leaves an error of at most
tol * max|f| / (alpha * min a); device and oracle both carry one."""

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import lib

TOL = 1e-9

CASES = [
    # extents, periodic, a, sigma, opts
    ((72, 72, 72), (False, False, False), False, 0.5, {}),
    ((36, 38, 34), (False, True, True), True, 0.5, dict(min_bottom_edge=16)),
    ((42, 46, 34), (True, True, True), True, 0.5, dict(min_bottom_edge=16, use_graph=0)),
    ((84, 68, 76), (True, False, False), False, 0.5, dict(min_bottom_edge=16)),
    ((66, 70, 58), (False, False, True), True, 0.5, dict(min_bottom_edge=20, coarse_tail=0)),
    ((52, 36, 44), (False, True, False), False, 2.0, dict(bottom_rel_tol=1e-8)),
    ((40, 44, 36), (False, False, False), True, 0.5, dict(nu1=1, nu2=1, min_bottom_edge=16)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("precision,krylov", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("ext,per,with_a,sigma,opts", CASES)
def test_solution_vs_oracle(ext, per, with_a, sigma, opts, precision, krylov):
    print(f"[deep] {ext} periodic {per} precision {precision} krylov {krylov} {opts}", flush=True)
    P = lib()
    rng = np.random.default_rng(7)
    dom = ((0, 0, 0), tuple(n - 1 for n in ext))
    boxes = [dom]
    opts = dict(dict(min_bottom_edge=18), **opts)
    plen = tuple(n / max(ext) for n in ext)
    alpha = 1.0
    bf = W.harmonic_faces(np.exp(sigma * rng.standard_normal(ext)), per)
    f = rng.uniform(-1.0, 1.0, ext)
    a = rng.uniform(0.5, 2.0, ext) if with_a else None
    fb = W.scatter_cells(f, boxes)
    b = [W.scatter_faces(bf[d], boxes, d) for d in range(3)]
    ab = W.scatter_cells(a, boxes) if with_a else None

    def mf(v, **kw):
        return P.MultiFab.from_numpy(boxes, v, **kw)

    bmf = [mf(b[d], ixtype=tuple(int(e == d) for e in range(3))) for d in range(3)]
    lev = O.make_level(boxes, dom, per, alpha, 1.0, ab, b, prob_len=plen)
    ophi = W.scatter_cells(np.zeros(ext), boxes, ng=1)
    O.pcg_solve(lev, ophi, fb, TOL, opts=O.Opts(symmetric=True))
    ref = W.gather_cells(ophi, boxes, ext, ng=1)
    bound = 2 * TOL * np.max(np.abs(f)) / (alpha * (a.min() if with_a else 1.0))
    s = P.MLMG(boxes, dom, per, alpha, 1.0, a=mf(ab) if with_a else None, b=bmf,
               opts=dict(tune=0, precision=precision, krylov=krylov, **opts), prob_hi=plen)
    for _ in range(2):  # the second solve replays what the first set up
        phi = mf(W.scatter_cells(np.zeros(ext), boxes, ng=1), ngrow=1)
        info = s.solve(phi, mf(fb), TOL)
        torch.cuda.synchronize()
        got = W.gather_cells(phi.valid_numpy(), boxes, ext, ng=0)
        assert np.max(np.abs(got - ref)) <= bound
        print("bottom iterations", info["bottom_iters"], "cycles", info["iters"], flush=True)
    s.close()
