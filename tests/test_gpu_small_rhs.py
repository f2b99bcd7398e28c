"""Solves of very small right-hand sides: the bottom CG's squared norms come
near the smallest numbers there, and the solve still takes the cycles of the
same right-hand side at scale 1 and gives its solution, scaled.  Each bottom CG:
one wavefront and one work-group, in the one-launch tail and alone, by runs of
cells, and preconditioned on a large bottom.

The scale is a power of two, so everything but the CG's scalars scales exactly.
Those lose bits once a square is subnormal (2^-1074 is the smallest), which
moves the bottom solves inside their own tolerance of 1e-4: the solution moves
by a small part of the residual tolerance times the condition of the operator,
1e-10 times at most 1e4 here."""

import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import lib

CASES = [
    # extents, opts
    ((32, 32, 32), {}),                            # 64 cells, in the tail
    ((40, 40, 40), {}),                            # 125 cells, in the tail
    ((32, 32, 32), dict(coarse_tail=0)),           # 64 cells alone
    ((36, 36, 36), dict(coarse_tail=0)),           # 729 cells alone
    ((48, 24, 32), dict(min_bottom_edge=12)),      # 24 x 12 x 16 cells, in runs
    ((72, 72, 72), dict(min_bottom_edge=18)),      # 18^3 cells, with coarsenings of their own
]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ext,opts", CASES)
def test_scaled_down_right_hand_side(ext, opts, precision):
    P = lib()
    rng = np.random.default_rng(11)
    dom = ((0, 0, 0), tuple(n - 1 for n in ext))
    boxes, per = [dom], (False, False, True)
    bf = W.harmonic_faces(np.exp(0.5 * rng.standard_normal(ext)), per)
    f = rng.uniform(-1.0, 1.0, ext)
    b = [P.MultiFab.from_numpy(boxes, W.scatter_faces(bf[d], boxes, d), 0,
                               ixtype=tuple(int(e == d) for e in range(3))) for d in range(3)]
    s = P.MLMG(boxes, dom, per, 0.0, 1.0, b=b, opts=dict(tune=0, precision=precision, **opts))
    out = []
    # FP32 cycles hold the residual itself in FP32, whose squares are far from
    # the smallest numbers of the FP64 scalars
    for e in (0, -60) if precision else (0, -480, -490):
        print(f"[small rhs] {ext} precision {precision} {opts} 2^{e}", flush=True)
        phi = s.cell_mf(1, fill=0.0)
        info = s.solve(phi, P.MultiFab.from_numpy(boxes, W.scatter_cells(np.ldexp(f, e), boxes), 0),
                       1e-10)
        torch.cuda.synchronize()
        out.append((info["iters"], np.ldexp(phi.valid_numpy()[0], -e)))
    s.close()
    ref = out[0]
    for it, x in out[1:]:
        assert it == ref[0]
        assert np.max(np.abs(x - ref[1])) <= 1e-6 * np.max(np.abs(ref[1]))
